// Compression kernels: dense filter bank -> CSR(C) (count, scan, ordered pack), the
// regrouping of the nonzeros into the (group, chunk, channel) stream the convolution
// kernel reads, dense activation -> per-pixel channel lists, and the helper max-pool.
//
// The paper (Sec. 3) fixes the format only: values, column indices and cumulative row
// counts that start with 0, one row per filter.  The construction used here is
// count -> exclusive scan -> order-preserving compaction, which makes the result unique
// (ascending flat index inside each row) and independent of thread scheduling.
#include <stddef.h>

#include "arrival.h"
#include "host_word.h"
#include "internal.h"

namespace fscnn {

namespace {

constexpr int kBlock = 256;

__device__ inline int lane_id() { return threadIdx.x & 63; }

// Stores that reach the memory that the XCDs' caches do not keep apart, and the last of a launch's work-groups to have made its own telling the
// host so: every stream finds them from there on.  (A wait for the stream is over 4 to 8 us later.)
template <class T> __device__ inline void store_through(T *p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// a wait for this wave's stores that the compiler moves nothing across either
__device__ inline void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
struct DeviceMem {
    __device__ int count(int *p, int most) const { return (int)atomicInc(reinterpret_cast<unsigned *>(p), (unsigned)most); }
};
__device__ inline bool arrived_last(int *counter) { return arrive(DeviceMem(), counter, (int)gridDim.x, (int)blockIdx.x); }
// a number for the host that waits for it
__device__ inline void store_host(int *p, int v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); }
// the same with the one behind it, at once: one store
__device__ inline void store_host(int *p, int v, int second)
{
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), (unsigned long long)(uint32_t)second << 32 | (uint32_t)v, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}
// the end of a kernel whose stores are all store_through(); counter NULL: nothing is told
__device__ inline void tell_host(int *counter, int *host)
{
    if (!counter) return;
    wait_stores();
    __syncthreads();
    if (threadIdx.x == 0 && arrived_last(counter)) store_host(host, 0);
}

// ---- exclusive scan of n ints into out[0..n] (out[n] = total); one work-group ---------
// Latency is all there is to it (n is a few thousand): a round takes up to 16 elements per thread,
// thread t the elements u*1024 + t, so that all its loads are coalesced and in flight together; every
// (u, wave) row of 64 is scanned with lane shuffles, the 256 row totals by the first wave, two barriers
// in all.  (A run of consecutive elements per thread and a scan of the 1024 sums with 20 barriers:
// 6.8 us on average over the 26 scans of loading the 13-layer stack.)
constexpr int kNoRow = 0x7fffffff;   // no row stores anything
// the smallest over a work-group, for all of it; part: an int per wave
template <int THREADS> __device__ inline int group_min(int v, int *part)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const int t = __shfl_xor(v, o, 64);
        v = t < v ? t : v;
    }
    if (lane_id() == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < THREADS / 64; ++i) v = part[i] < v ? part[i] : v;
    return v;
}
constexpr int kScanThreads = 1024, kScanPer = 16, kScanRows = kScanThreads / 64 * kScanPer;
__device__ inline int wave_inclusive(int v)
{
    const int lane = lane_id();
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(v, o, 64);
        if (lane >= o) v += t;
    }
    return v;
}
__global__ void __launch_bounds__(kScanThreads) exclusive_scan_kernel(const int *__restrict__ in,
                                                                      int *__restrict__ out,
                                                                      long long n, int *__restrict__ host, int fewest)
{
    __shared__ int rows[kScanRows + 1];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    int carry = 0, few = kNoRow;
    for (long long n0 = 0; n0 < n; n0 += kScanThreads * kScanPer) {
        int v[kScanPer], incl[kScanPer];
        const long long left = n - n0;
#pragma unroll
        for (int u = 0; u < kScanPer; ++u) {
            const int i = u * kScanThreads + (int)threadIdx.x;
            v[u] = i < left ? in[n0 + i] : 0;
        }
#pragma unroll
        for (int u = 0; u < kScanPer; ++u) few = v[u] > 0 && v[u] < few ? v[u] : few;
#pragma unroll
        for (int u = 0; u < kScanPer; ++u) {
            incl[u] = 0;
            if ((long long)u * kScanThreads < left) incl[u] = wave_inclusive(v[u]);   // (the same for the whole group)
            if (lane == 63) rows[u * (kScanThreads / 64) + wave] = incl[u];
        }
        __syncthreads();
        if (wave == 0) {
            constexpr int Q = kScanRows / 64;
            int t[Q], s = 0;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                t[q] = s;
                s += rows[lane * Q + q];
            }
            const int end = wave_inclusive(s);
#pragma unroll
            for (int q = 0; q < Q; ++q) rows[lane * Q + q] = end - s + t[q];
            if (lane == 63) rows[kScanRows] = end;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kScanPer; ++u) {
            const int i = u * kScanThreads + (int)threadIdx.x;
            if (i < left) out[n0 + i] = carry + rows[u * (kScanThreads / 64) + wave] + incl[u] - v[u];
        }
        carry += rows[kScanRows];
        __syncthreads();   // the next round writes `rows`
    }
    if (fewest) few = group_min<kScanThreads>(few, rows);
    if (threadIdx.x == 0) {
        out[n] = carry;
        if (fewest) out[n + 1] = few;
        if (host && fewest) store_host(host, carry, few);
        else if (host) store_host(host, carry);
    }
}

// the smallest of in[] above 0, where no work-group that scans sees all of it
__global__ void __launch_bounds__(kScanThreads) scan_fewest_kernel(const int *__restrict__ in, long long n, int *__restrict__ out, int *__restrict__ host)
{
    __shared__ int part[kScanThreads / 64];
    int few = kNoRow;
    for (long long n0 = threadIdx.x; n0 < n; n0 += kScanThreads * kScanPer) {
        int v[kScanPer];
#pragma unroll
        for (int u = 0; u < kScanPer; ++u) v[u] = n0 + u * kScanThreads < n ? in[n0 + u * kScanThreads] : 0;
#pragma unroll
        for (int u = 0; u < kScanPer; ++u) few = v[u] > 0 && v[u] < few ? v[u] : few;
    }
    few = group_min<kScanThreads>(few, part);
    if (threadIdx.x == 0) {
        *out = few;
        if (host) store_host(host, few);
    }
}

// ---- the same for large n, three passes over tiles of kTile elements -------------------
// (1) every work-group adds up its tile; (2) the tile sums are scanned by the single-group
// kernel above; (3) every work-group scans its tile starting from its tile's offset.  Tiles go
// through LDS so that global loads and stores are contiguous while each thread scans a
// contiguous run.
constexpr int kTileThreads = 256, kTilePer = 16, kTile = kTileThreads * kTilePer;

__global__ void __launch_bounds__(kTileThreads) scan_tile_sum_kernel(const int *__restrict__ in,
                                                                     long long n, int *__restrict__ tsum)
{
    __shared__ int part[kTileThreads / 64];
    const long long base = (long long)blockIdx.x * kTile;
    int s = 0;
#pragma unroll
    for (int k = 0; k < kTilePer; ++k) {
        const long long i = base + k * kTileThreads + threadIdx.x;
        if (i < n) s += in[i];
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
    if (lane_id() == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int i = 0; i < kTileThreads / 64; ++i) t += part[i];
        tsum[blockIdx.x] = t;
    }
}

__global__ void __launch_bounds__(kTileThreads) scan_tile_kernel(const int *__restrict__ in, long long n,
                                                                 const int *__restrict__ toff,
                                                                 int *__restrict__ out)
{
    __shared__ int tile[kTile + kTile / 32];     // padded: a thread's run of 16 starts in its own bank group
    __shared__ int tsum[kTileThreads];
    const long long base = (long long)blockIdx.x * kTile;
    auto at = [](int e) { return e + e / 32; };
#pragma unroll
    for (int k = 0; k < kTilePer; ++k) {
        const int e = k * kTileThreads + threadIdx.x;
        tile[at(e)] = base + e < n ? in[base + e] : 0;
    }
    __syncthreads();
    int s = 0;
#pragma unroll
    for (int k = 0; k < kTilePer; ++k) s += tile[at(threadIdx.x * kTilePer + k)];
    tsum[threadIdx.x] = s;
    __syncthreads();
    for (int o = 1; o < kTileThreads; o <<= 1) {
        const int v = (int)threadIdx.x >= o ? tsum[threadIdx.x - o] : 0;
        __syncthreads();
        tsum[threadIdx.x] += v;
        __syncthreads();
    }
    int run = toff[blockIdx.x] + (threadIdx.x == 0 ? 0 : tsum[threadIdx.x - 1]);
#pragma unroll
    for (int k = 0; k < kTilePer; ++k) {
        const int idx = at(threadIdx.x * kTilePer + k);
        const int v = tile[idx];
        tile[idx] = run;
        run += v;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kTilePer; ++k) {
        const int e = k * kTileThreads + threadIdx.x;
        if (base + e < n) out[base + e] = tile[at(e)];
    }
    // the grand total goes to out[n]
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == kTileThreads - 1) out[n] = toff[gridDim.x];
}

__device__ int g_count_slots[HostWord::kWords * kCounterInts];
constexpr int kCountScan = 4096;   // rows that one work-group scans

// ---- A1: per output channel, the number of entries with w != 0 ------------------------
// With a counter the work-group that finishes last scans the counts as well (rowptr, and the total and the fewest for the host): the scan as a launch of
// its own was 3.4 us and the gap in front of it.
// (a 512 x 3 x 3 row is one round: the bank's 9.4 MB, counted and scanned, take 13.9 us in two rounds of 256 threads with one counter, 8.6 so)
constexpr int kCountThreads = 512, kCountPer = 9;
__global__ void __launch_bounds__(kCountThreads) filter_count_kernel(const float *__restrict__ w, long long row, int *__restrict__ cnt,
                                                              int *__restrict__ rowptr, int *__restrict__ counter, int *__restrict__ host)
{
    __shared__ int part[kCountThreads / 64], last;
    const float *wk = w + (long long)blockIdx.x * row;
    int c = 0;
    for (long long f = threadIdx.x; f < row; f += kCountThreads * kCountPer) {   // all loads of a round in flight together
        float v[kCountPer];
#pragma unroll
        for (int u = 0; u < kCountPer; ++u) v[u] = f + u * kCountThreads < row ? wk[f + u * kCountThreads] : 0.0f;
#pragma unroll
        for (int u = 0; u < kCountPer; ++u) c += (v[u] != 0.0f) ? 1 : 0;
    }
    for (int o = 32; o > 0; o >>= 1) c += __shfl_down(c, o, 64);
    if (lane_id() == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int i = 0; i < kCountThreads / 64; ++i) t += part[i];
        store_through(cnt + blockIdx.x, t);
        wait_stores();
        last = counter && arrived_last(counter);
    }
    __syncthreads();
    if (!last) return;
    const int K = (int)gridDim.x, wave = threadIdx.x >> 6;
    int carry = 0, few = kNoRow;
    for (int k0 = 0; k0 < K; k0 += kCountThreads) {
        const int k = k0 + (int)threadIdx.x;
        const int v = k < K ? __hip_atomic_load(cnt + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
        few = v > 0 && v < few ? v : few;
        const int incl = wave_inclusive(v);
        if (lane_id() == 63) part[wave] = incl;
        __syncthreads();
        int before = carry;
#pragma unroll
        for (int i = 0; i < kCountThreads / 64; ++i) {
            if (i < wave) before += part[i];
            carry += part[i];
        }
        if (k < K) rowptr[k] = before + incl - v;
        __syncthreads();   // the next round writes `part`
    }
    few = group_min<kCountThreads>(few, part);
    if (threadIdx.x == 0) {
        rowptr[K] = carry;
        rowptr[K + 1] = few;
        if (host) store_host(host, carry, few);
    }
}

// ---- A2: ordered pack of row k into idx/val at rowptr[k] ------------------------------
// A round takes kPackPer elements per thread, a wave 64 * kPackPer consecutive ones: all loads in flight
// together, positions by ballots, one exchange of the wave totals (one element per thread and round, two
// barriers each, spent its time in the 18 rounds of a 512 x 3 x 3 row).
constexpr int kPackThreads = 512, kPackPer = 9;   // (again one round for 512 x 3 x 3)
__global__ void __launch_bounds__(kPackThreads) filter_pack_kernel(const float *__restrict__ w,
                                                             long long row,
                                                             const int *__restrict__ rowptr,
                                                             uint32_t *__restrict__ idx,
                                                             float *__restrict__ val, int *__restrict__ counter, int *__restrict__ host)
{
    __shared__ int wave_tot[2][kPackThreads / 64];
    const int k = blockIdx.x, lane = lane_id(), wave = threadIdx.x >> 6;
    const float *wk = w + (long long)k * row;
    long long base = rowptr[k];
    int side = 0;
    for (long long f0 = 0; f0 < row; f0 += kPackThreads * kPackPer) {
        const long long first = f0 + wave * (64 * kPackPer) + lane;
        float v[kPackPer];
#pragma unroll
        for (int u = 0; u < kPackPer; ++u) v[u] = first + u * 64 < row ? wk[first + u * 64] : 0.0f;
        int pos[kPackPer], tot = 0;
#pragma unroll
        for (int u = 0; u < kPackPer; ++u) {
            const unsigned long long m = __ballot(v[u] != 0.0f);
            pos[u] = tot + __popcll(m & ((1ull << lane) - 1ull));
            tot += __popcll(m);
        }
        if (lane == 0) wave_tot[side][wave] = tot;
        __syncthreads();
        long long at = base;
#pragma unroll
        for (int i = 0; i < kPackThreads / 64; ++i) {
            const int t = wave_tot[side][i];
            if (i < wave) at += t;
            base += t;
        }
        side ^= 1;   // the next round's totals go to the other set: one barrier per round is enough
#pragma unroll
        for (int u = 0; u < kPackPer; ++u)
            if (v[u] != 0.0f) {
                store_through(idx + at + pos[u], (uint32_t)(first + u * 64));
                store_through(val + at + pos[u], v[u]);
            }
    }
    tell_host(counter, host);
}

// ---- A3: regroup into (group g, chunk ci, channel-in-group kk) buckets -----------------
// Rows are ascending in the flat index, hence ascending in c: the entries of chunk ci are the
// contiguous run with ci*CC*R*S <= flat < (ci+1)*CC*R*S, found by binary search.
__device__ inline int lower_bound_u32(const uint32_t *a, int lo, int hi, uint32_t key)
{
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] < key) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// Bucket (group g, wave w, chunk ci, slot j), slot fastest: the records of one wave form one contiguous stream ordered by (chunk,
// slot); its output channel is k = g*KG + w*SLOTS + j.  A wave's channels are SLOTS adjacent rows, so its stream starts where the
// first of them does and nothing has to be counted across waves: a work-group builds a wave's stream whole.  It reads the rows' entries
// twice, all loads coalesced: first for where the chunks begin (an entry whose chunk is not the one of the entry before), then,
// after a scan over the buckets, to write the records.  Three launches before (count by bisection, scan, fill): 5.5 + 3.4 + 5.4 us and the
// gaps between them on average over the stack's layers, one of 6.9 us now, of which 1.3 are for
// stores and arrivals that end the host's wait early.
// mem: where the chunks' first entries go if they do not fit the LDS (lds_ints); recs may be NULL (only the pointers are wanted)
__global__ void __launch_bounds__(kBlock) plan_kernel(const int *__restrict__ rowptr, const uint32_t *__restrict__ idx,
                                                      const float *__restrict__ val, int K, int R, int S, int CC, int SLOTS, int NCH,
                                                      int IN_ROWS, int PITCH, int BV, int STRIDE, int nwaves, int lds_ints,
                                                      int *__restrict__ mem, int *__restrict__ segptr, Rec *__restrict__ recs,
                                                      int *__restrict__ counter, int *__restrict__ host)
{
    extern __shared__ int plan_lds[];
    __shared__ int part[kBlock / 64];
    const int gw = blockIdx.x, RS = R * S, wave = threadIdx.x >> 6, B = NCH * SLOTS;
    const uint32_t per = (uint32_t)(CC * RS);
    // first entry of chunk c of row j: at[j * (NCH + 1) + c], the row's end at c = NCH; then every bucket's first record
    const bool fits = 2 * B + SLOTS <= lds_ints;
    int *at = fits ? plan_lds : mem + (long long)gw * (2 * B + SLOTS), *seg = at + SLOTS * (NCH + 1);
    const int k0 = gw * SLOTS;
    auto row = [&](int k) { return rowptr[k < K ? k : K]; };
    const int base = row(k0);
    for (int j = 0; j < SLOTS; ++j) {
        int *a = at + j * (NCH + 1);
        const int lo = row(k0 + j), hi = row(k0 + j + 1);
        for (int i = lo + (int)threadIdx.x; i <= hi; i += kBlock) {      // (hi: behind the last entry)
            const int c = i < hi ? (int)(idx[i] / per) : NCH, p = i > lo ? (int)(idx[i - 1] / per) : -1;
            for (int q = p + 1; q <= c; ++q) a[q] = i;
        }
    }
    __syncthreads();
    int *out = segptr + (long long)gw * B;
    int carry = base;
    for (int b0 = 0; b0 < B; b0 += kBlock) {
        const int b = b0 + (int)threadIdx.x;
        int v = 0;
        if (b < B) {
            const int *a = at + (b % SLOTS) * (NCH + 1) + b / SLOTS;
            v = a[1] - a[0];
        }
        const int incl = wave_inclusive(v);
        if (lane_id() == 63) part[wave] = incl;
        __syncthreads();
        int before = carry;
#pragma unroll
        for (int i = 0; i < kBlock / 64; ++i) {
            if (i < wave) before += part[i];
            carry += part[i];
        }
        if (b < B) store_through(out + b, seg[b] = before + incl - v);
        __syncthreads();   // the next round writes `part`
    }
    if (gw == nwaves - 1 && threadIdx.x == 0) store_through(out + B, carry);
    if (!recs) return;                                // (another launch follows)
    // a record is one 64-bit number
    auto put = [&](long long at, uint32_t off, float val) {
        store_through(reinterpret_cast<unsigned long long *>(recs) + at, (unsigned long long)__float_as_uint(val) << 32 | off);
    };
    if (gw == nwaves - 1 && (int)threadIdx.x < kPlanSpare) put(carry + (int)threadIdx.x, 0u, 0.0f);   // spare records that a prefetching reader may touch past the end
    for (int j = 0; j < SLOTS; ++j) {
        const int *a = at + j * (NCH + 1);
        const int lo = row(k0 + j), hi = row(k0 + j + 1);
        for (int i = lo + (int)threadIdx.x; i < hi; i += kBlock) {
            const uint32_t f = idx[i];
            const int ci = (int)(f / per), c = (int)(f / RS) - ci * CC;
            const int rs = (int)(f % RS);
            const int r = rs / S, s = rs % S;
            // stride 2: tap (r, s) lies in plane (r mod 2, s mod 2) of the channel at (r/2, s/2)
            const int plane = (r % STRIDE) * STRIDE + (s % STRIDE);
            put(seg[ci * SLOTS + j] + i - a[ci],
                (uint32_t)(((((c * STRIDE * STRIDE + plane) * IN_ROWS) + r / STRIDE) * PITCH + s / STRIDE) * BV * 4), val[i]);
        }
    }
    tell_host(counter, host);
}
static_assert(sizeof(Rec) == 8 && offsetof(Rec, off) == 0, "written as one number");

// The plan of the taps-outer form: for every (group, wave, chunk), CC*R*S groups of SLOTS records
// {LDS byte offset of tap (c mod CC, r, s), weight of output channel (group*WAVES + wave)*SLOTS + j
// at that tap}, a zero weight where the row stores nothing there (or k, c lie past the bank).
__global__ void plan_fill_dense_kernel(const int *__restrict__ rowptr, const uint32_t *__restrict__ idx,
                                       const float *__restrict__ val, int K, int C, int R, int S, int CC,
                                       int SLOTS, int WAVES, int NCH, int NG, int IN_ROWS, int PITCH,
                                       int BV, long long nrec, Rec *__restrict__ recs)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kPlanSpare) {
        Rec z;
        z.off = 0u;
        z.val = 0.0f;
        recs[nrec + i] = z;
    }
    if (i >= nrec) return;
    const int RS = R * S, T = CC * RS;
    const int j = (int)(i % SLOTS);
    const int t = (int)((i / SLOTS) % T);
    const int ci = (int)((i / ((long long)SLOTS * T)) % NCH);
    const long long gw = i / ((long long)SLOTS * T * NCH);   // group * WAVES + wave
    const int k = (int)(gw * SLOTS + j);
    const int cl = t / RS, rs = t % RS;
    const int c = ci * CC + cl;
    Rec rec;
    rec.off = (uint32_t)((((cl * IN_ROWS) + rs / S) * PITCH + rs % S) * BV * 4);
    rec.val = 0.0f;
    if (k < K && c < C) {
        const uint32_t flat = (uint32_t)(c * RS + rs);
        const int lo = rowptr[k], hi = rowptr[k + 1];
        const int at = lower_bound_u32(idx, lo, hi, flat);
        if (at < hi && idx[at] == flat) rec.val = val[at];
    }
    recs[i] = rec;
}

// ---- A7: compressed activation, rows = pixels, columns = channels ----------------------
// A work-group owns PX consecutive pixels (PX a power of two, at most 32), whose lists are adjacent in
// memory.  (1) The stored values of every group are counted; (2) a scan of these few sums gives where a
// group's lists start; (3) the group counts again per (pixel, step of CC channels), scans that in LDS --
// the chunk pointers the convolution kernels read, at step 0 the start of the pixel's row -- and writes
// pointers and lists.  The activation is read twice, from the last-level cache the second time; nothing
// else goes through memory.  (Counts per (pixel, step) written out and scanned there, 401 000 of them for
// 8 x 512 x 28 x 28, were four launches and 29 us in front of step 3.)

// with cnt: the counts per (pixel, step) are at hand (sparse output emission) and are only added up
template <int BLOCK>
__global__ void __launch_bounds__(BLOCK) input_sum_kernel(const float *__restrict__ x, const int *__restrict__ cnt,
                                                           int C, long long HW, long long npix, int NCH, int PX,
                                                           int *__restrict__ sums)
{
    __shared__ int part[BLOCK / 64];
    const long long p0 = (long long)blockIdx.x * PX, p1 = p0 + PX < npix ? p0 + PX : npix;
    int c = 0;
    if (cnt) {
        const int m = (int)(p1 - p0) * NCH;
        for (int i = threadIdx.x; i < m; i += BLOCK) c += cnt[p0 * NCH + i];
    } else {
        const long long p = p0 + threadIdx.x % PX;
        const int step = BLOCK / PX;
        if (p < npix) {
            const float *xp = x + p / HW * C * HW + p % HW;
            for (int ch = threadIdx.x / PX; ch < C; ch += 16 * step) {   // sixteen loads in flight
                float v[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) v[u] = ch + u * step < C ? xp[(long long)(ch + u * step) * HW] : 0.0f;
#pragma unroll
                for (int u = 0; u < 16; ++u) c += v[u] != 0.0f ? 1 : 0;
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) c += __shfl_down(c, o, 64);
    if (lane_id() == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int i = 0; i < BLOCK / 64; ++i) t += part[i];
        sums[blockIdx.x] = t;
    }
}

// Thread (pixel px, step lane sj) walks the steps sj, sj + 256/PX, ... of its pixel, so the reads of a
// channel plane cover PX adjacent floats; the values of its kKept steps stay in registers between
// counting and placing (PX * NCH <= BLOCK * kKept).  The (channel, value) pairs meet in an LDS image of the group's output range,
// copied out with fully coalesced stores.
template <int BLOCK, int kKept>
__global__ void __launch_bounds__(BLOCK) input_fill_kernel(const float *__restrict__ x, int C, long long HW,
                                                            long long npix, int NCH, int PX,
                                                            int *__restrict__ start, const int *__restrict__ sums,
                                                            int *__restrict__ cptr,
                                                            uint32_t *__restrict__ cidx, float *__restrict__ xval,
                                                            int spare, float *__restrict__ dense, int dense_from, int *__restrict__ host)
{
    constexpr int CC = kSiCC;
    extern __shared__ uint32_t stage[];   // [cap] value bit patterns, then in 16 bits [cap] channels, [PX * NCH] positions
    __shared__ int wave_sum[BLOCK / 64], wave_all[BLOCK / 64];
    const int cap = PX * NCH * CC, M = PX * NCH;
    unsigned short *chan = reinterpret_cast<unsigned short *>(stage + cap), *pos = chan + cap;   // (cap is below 10500)
    const long long p0 = (long long)blockIdx.x * PX;
    const int px = threadIdx.x % PX, sj = threadIdx.x / PX, SJ = BLOCK / PX;
    const long long p = p0 + px;
    const bool live = p < npix;
    const long long first = live ? p / HW * C * HW + p % HW : 0;
    const float *xp = x + first;
    auto load = [&](int j, float(&v)[CC]) {
#pragma unroll
        for (int u = 0; u < CC; ++u) {
            const int ch = j * CC + u;
            v[u] = live && j < NCH && ch < C ? xp[(long long)ch * HW] : 0.0f;
        }
    };
    float kept[kKept][CC];
#pragma unroll
    for (int r = 0; r < kKept; ++r) load(sj + r * SJ, kept[r]);
    // where the lists start and how many values there are in all: as scanned, or (sums) added up here
    int base, all;
    if (!sums) {
        base = start[blockIdx.x];
        all = start[gridDim.x];
    } else {
        int before = 0, every = 0;
        for (int i = threadIdx.x; i < (int)gridDim.x; i += BLOCK) {
            const int v = sums[i];
            every += v;
            before += i < (int)blockIdx.x ? v : 0;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            before += __shfl_down(before, o, 64);
            every += __shfl_down(every, o, 64);
        }
        if (lane_id() == 0) {
            wave_sum[threadIdx.x >> 6] = before;
            wave_all[threadIdx.x >> 6] = every;
        }
        __syncthreads();
        base = all = 0;
#pragma unroll
        for (int i = 0; i < BLOCK / 64; ++i) {
            base += wave_sum[i];
            all += wave_all[i];
        }
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            start[gridDim.x] = all;
            if (host) store_host(host, all);
        }
    }
    // the entries past the last stored one (readers fetch a few positions ahead) and the last pointer
    if (blockIdx.x == 0 && (int)threadIdx.x <= spare) {
        if ((int)threadIdx.x == spare) {
            cptr[npix * NCH] = all;
        } else {
            cidx[all + threadIdx.x] = 0u;
            xval[all + threadIdx.x] = 0.0f;
        }
    }
    float *dp = live && dense && all >= dense_from ? dense + first : nullptr;
    auto count = [&](int j, const float(&v)[CC]) {
        if (dp) {
#pragma unroll
            for (int u = 0; u < CC; ++u) {
                const int ch = j * CC + u;
                if (j < NCH && ch < C) dp[(long long)ch * HW] = v[u];
            }
        }
        int c = 0;
#pragma unroll
        for (int u = 0; u < CC; ++u) c += v[u] != 0.0f ? 1 : 0;
        if (j < NCH) pos[px * NCH + j] = (unsigned short)c;
    };
    auto place = [&](int j, const float(&v)[CC]) {
        int o = j < NCH ? pos[px * NCH + j] : 0;
#pragma unroll
        for (int u = 0; u < CC; ++u)
            if (v[u] != 0.0f) {
                chan[o] = (unsigned short)(j * CC + u);
                stage[o] = __float_as_uint(v[u]);
                ++o;
            }
    };
#pragma unroll
    for (int r = 0; r < kKept; ++r) count(sj + r * SJ, kept[r]);
    __syncthreads();
    // counts -> positions in the group's range: a run of them per thread
    const int per = (M + BLOCK - 1) / BLOCK, a = (int)threadIdx.x * per, b = a + per < M ? a + per : M;
    int s = 0;
    for (int i = a; i < b; ++i) s += pos[i];
    const int incl = wave_inclusive(s);
    if (lane_id() == 63) wave_sum[threadIdx.x >> 6] = incl;
    __syncthreads();
    int run = incl - s, total = 0;
#pragma unroll
    for (int i = 0; i < BLOCK / 64; ++i) {
        if (i < (int)(threadIdx.x >> 6)) run += wave_sum[i];
        total += wave_sum[i];
    }
    for (int i = a; i < b; ++i) {
        const int c = pos[i];
        pos[i] = (unsigned short)run;
        run += c;
    }
    __syncthreads();
    const int m = (int)((p0 + PX < npix ? p0 + PX : npix) - p0) * NCH;
    for (int i = threadIdx.x; i < m; i += BLOCK) cptr[p0 * NCH + i] = base + pos[i];
#pragma unroll
    for (int r = 0; r < kKept; ++r) place(sj + r * SJ, kept[r]);
    __syncthreads();
    for (int t = threadIdx.x; t < total; t += BLOCK) {
        cidx[base + t] = chan[t];
        xval[base + t] = __uint_as_float(stage[t]);
    }
}

// ---- helper: 2x2 / stride-2 max pooling ------------------------------------------------
__global__ void __launch_bounds__(kBlock) maxpool2x2_kernel(const float *__restrict__ x,
                                                            long long NC, int H, int W, int Ho,
                                                            int Wo, float *__restrict__ y)
{
    const long long o = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (o >= NC * Ho * Wo) return;
    const int ox = (int)(o % Wo);
    const int oy = (int)((o / Wo) % Ho);
    const long long nc = o / ((long long)Wo * Ho);
    const float *p = x + (nc * H + 2 * oy) * W + 2 * ox;
    float m = p[0];
    m = p[1] > m ? p[1] : m;
    m = p[W] > m ? p[W] : m;
    m = p[W + 1] > m ? p[W + 1] : m;
    y[o] = m;
}

// same pooling on a batch-interleaved (N4) tensor: one thread per output pixel of one image
// group, all four images at once
__global__ void __launch_bounds__(kBlock) maxpool2x2_n4_kernel(const float4 *__restrict__ x,
                                                               long long GC, int H, int W, int Ho,
                                                               int Wo, float4 *__restrict__ y)
{
    const long long o = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (o >= GC * Ho * Wo) return;
    const int ox = (int)(o % Wo);
    const int oy = (int)((o / Wo) % Ho);
    const long long gc = o / ((long long)Wo * Ho);
    const float4 *p = x + (gc * H + 2 * oy) * W + 2 * ox;
    const float4 a = p[0], b = p[1], c = p[W], d = p[W + 1];
    auto mx4 = [](float p0, float p1, float p2, float p3) {  // same compare order as the NCHW kernel
        float m = p0;
        m = p1 > m ? p1 : m;
        m = p2 > m ? p2 : m;
        m = p3 > m ? p3 : m;
        return m;
    };
    y[o] = make_float4(mx4(a.x, b.x, c.x, d.x), mx4(a.y, b.y, c.y, d.y), mx4(a.z, b.z, c.z, d.z),
                       mx4(a.w, b.w, c.w, d.w));
}

// NCHW <-> N4 ([ceil(N/4)][C][H][W][4]); images past N read as / are written as nothing (N4 pad
// lanes are filled with 0)
__global__ void __launch_bounds__(kBlock) layout_convert_kernel(const float *__restrict__ src,
                                                                int N, long long CHW, int src_n4,
                                                                float *__restrict__ dst)
{
    const long long t = (long long)blockIdx.x * kBlock + threadIdx.x;
    const long long groups = (N + 3) / 4;
    if (t >= groups * CHW) return;
    const long long g = t / CHW, q = t % CHW;
    if (src_n4) {
        const float4 v = reinterpret_cast<const float4 *>(src)[t];
        const float e[4] = {v.x, v.y, v.z, v.w};
        for (int b = 0; b < 4; ++b)
            if (g * 4 + b < N) dst[(g * 4 + b) * CHW + q] = e[b];
    } else {
        float e[4];
        for (int b = 0; b < 4; ++b) e[b] = g * 4 + b < N ? src[(g * 4 + b) * CHW + q] : 0.0f;
        reinterpret_cast<float4 *>(dst)[t] = make_float4(e[0], e[1], e[2], e[3]);
    }
}

inline unsigned blocks_for(long long n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

// The counter, on the current device, of a launch that writes the host's word of this slot; none (NULL) for slot -1
static hipError_t count_slot(int slot, int **p)
{
    *p = nullptr;
    if (slot < 0) return hipSuccess;
    constexpr int kDevices = 64;
    static std::atomic<int *> known[kDevices];
    int dev;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    int *q = dev < kDevices ? known[dev].load() : nullptr;
    if (!q) {
        e = hipGetSymbolAddress(reinterpret_cast<void **>(&q), HIP_SYMBOL(g_count_slots));
        if (e == hipSuccess && dev < kDevices) known[dev] = q;
    }
    *p = q + slot * kCounterInts;
    return e;
}

long long scan_tmp_elems(long long n)
{
    return n <= 4 * kTile ? 0 : 2 * ((n + kTile - 1) / kTile) + 2;
}

hipError_t launch_exclusive_scan(const int *in, int *out, long long n, int *tmp, int *host, bool fewest, hipStream_t st)
{
    if (n <= 4 * kTile) {
        hipLaunchKernelGGL(exclusive_scan_kernel, dim3(1), dim3(kScanThreads), 0, st, in, out, n, host, fewest ? 1 : 0);
        return hipGetLastError();
    }
    const long long nt = (n + kTile - 1) / kTile;
    int *tsum = tmp, *toff = tmp + nt;   // toff has nt + 1 entries
    hipLaunchKernelGGL(scan_tile_sum_kernel, dim3((unsigned)nt), dim3(kTileThreads), 0, st, in, n, tsum);
    if (fewest) hipLaunchKernelGGL(scan_fewest_kernel, dim3(1), dim3(kScanThreads), 0, st, in, n, out + n + 1, host ? host + 1 : nullptr);
    hipLaunchKernelGGL(exclusive_scan_kernel, dim3(1), dim3(kScanThreads), 0, st, tsum, toff, nt, host, 0);
    hipLaunchKernelGGL(scan_tile_kernel, dim3((unsigned)nt), dim3(kTileThreads), 0, st, in, n, toff, out);
    return hipGetLastError();
}

hipError_t launch_filter_count(const float *w, int K, long long row, int *cnt, int *rowptr, int slot, int *host, hipStream_t st)
{
    int *counter = nullptr;
    const hipError_t ce = count_slot(K <= kCountScan ? slot : -1, &counter);
    if (ce != hipSuccess) return ce;
    hipLaunchKernelGGL(filter_count_kernel, dim3(K), dim3(kCountThreads), 0, st, w, row, cnt, rowptr, counter, host);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess || counter ? e : launch_exclusive_scan(cnt, rowptr, K, cnt + K, host, true, st);
}

hipError_t launch_filter_pack(const float *w, int K, long long row, const int *rowptr,
                              uint32_t *idx, float *val, int slot, int *host, hipStream_t st)
{
    int *counter = nullptr;
    const hipError_t e = count_slot(slot, &counter);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(filter_pack_kernel, dim3(K), dim3(kPackThreads), 0, st, w, row, rowptr, idx, val, counter, host);
    return hipGetLastError();
}

constexpr int kPlanLds = 12288;   // ints
long long plan_scratch_elems(const SfGeom &g, int NCH, int NG)
{
    const long long per = 2LL * NCH * g.SLOTS + g.SLOTS;
    return per <= kPlanLds ? 0 : per * NG * g.WAVES;
}

hipError_t launch_plan(const int *rowptr, const uint32_t *idx, const float *val, int K, int R, int S, const SfGeom &g, int NCH, int NG,
                       int *scratch, int *segptr, Rec *recs, int slot, int *host, hipStream_t st)
{
    int *counter = nullptr;
    const hipError_t e = count_slot(slot, &counter);
    if (e != hipSuccess) return e;
    const long long waves = (long long)NG * g.WAVES, per = 2LL * NCH * g.SLOTS + g.SLOTS;
    const size_t lds = per <= kPlanLds ? sizeof(int) * (size_t)per : 0;
    hipLaunchKernelGGL(plan_kernel, dim3((unsigned)waves), dim3(kBlock), lds, st, rowptr, idx, val, K, R, S, g.CC, g.SLOTS, NCH, g.IN_ROWS,
                       g.PITCH, g.BV, g.STRIDE, (int)waves, lds ? kPlanLds : 0, scratch, segptr, recs, counter, host);
    return hipGetLastError();
}

hipError_t launch_plan_fill_dense(const int *rowptr, const uint32_t *idx, const float *val, int K, int C,
                                  int R, int S, const SfGeom &g, int NCH, int NG, long long nrec, Rec *recs,
                                  hipStream_t st)
{
    const long long n = nrec > kPlanSpare ? nrec : kPlanSpare;
    hipLaunchKernelGGL(plan_fill_dense_kernel, dim3(blocks_for(n, kBlock)), dim3(kBlock), 0, st, rowptr, idx,
                       val, K, C, R, S, g.CC, g.SLOTS, g.WAVES, NCH, NG, g.IN_ROWS, g.PITCH, g.BV, nrec, recs);
    return hipGetLastError();
}

// LDS bytes of the fill pass per pixel and step: 6 per possible entry, 2 for its position
constexpr int kFillBytes = kSiCC * 6 + 2;
// pixels per work-group: as many (up to 32) as fit 64 KB; 0: too many channels, not served
static int input_pixels(int NCH)
{
    int PX = 32;
    while (PX > 0 && (long long)PX * NCH * kFillBytes > 65536) PX /= 2;
    return PX;
}

long long input_groups(long long npix, int NCH)
{
    const int PX = input_pixels(NCH);
    return PX ? (npix + PX - 1) / PX : 0;
}

// Up to as many groups every work-group of the fill pass adds up the groups before its own (a few loads per thread, behind those of x)
// instead of a scan between the passes (8 x 512 x 28 x 28, 784 groups: 0.9 us here, 3.6 and the gap as a launch; 2 x 87 x 31 x 38 compressed
// and convolved: 46.0 us with the scan, 42.0)
constexpr long long kFillSums = 2048;
bool input_scans(long long npix, int NCH) { return input_groups(npix, NCH) > kFillSums; }

long long input_scratch_elems(long long npix, int NCH)
{
    const long long g = input_groups(npix, NCH);
    return 2 * g + 1 + scan_tmp_elems(g);
}

hipError_t launch_input_sums(const float *x, const int *cnt, int N, int C, int H, int W, int NCH, int *scratch, bool scan,
                             int *host, hipStream_t st)
{
    const long long HW = (long long)H * W, npix = (long long)N * HW, g = input_groups(npix, NCH);
    if (g == 0) return hipErrorInvalidValue;
    const int PX = input_pixels(NCH);
    // a pass over x is latency and loads in flight: 16 waves per group from four values per thread on (8 x 512 x 28 x 28: 13.5 us with
    // four waves, 6.5); counts at hand are few
    if (!cnt && C * PX >= 4096)
        hipLaunchKernelGGL(input_sum_kernel<1024>, dim3((unsigned)g), dim3(1024), 0, st, x, cnt, C, HW, npix, NCH, PX, scratch + g + 1);
    else
        hipLaunchKernelGGL(input_sum_kernel<256>, dim3((unsigned)g), dim3(256), 0, st, x, cnt, C, HW, npix, NCH, PX, scratch + g + 1);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess || !scan ? e : launch_exclusive_scan(scratch + g + 1, scratch, g, scratch + 2 * g + 1, host, false, st);
}

hipError_t launch_input_fill(const float *x, int N, int C, int H, int W, int NCH, int *scratch, bool scanned, int *cptr,
                             uint32_t *cidx, float *xval, int spare, float *dense, long long dense_from, int *host, hipStream_t st)
{
    const long long HW = (long long)H * W, npix = (long long)N * HW, g = input_groups(npix, NCH);
    if (g == 0 || spare >= kBlock) return hipErrorInvalidValue;
    const int PX = input_pixels(NCH);
    const size_t lds = (size_t)PX * NCH * kFillBytes;
    auto launch = [&](auto kernel, int block) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)g), dim3(block), lds, st, x, C, HW, npix, NCH, PX, scratch, scanned ? nullptr : scratch + g + 1, cptr, cidx,
                           xval, spare, dense, (int)dense_from, host);
    };
    // Two to three steps per thread, all kept: 512 threads where there are steps for more than 256 (8 x 512 x 28 x 28, dense form
    // included: 16.0 us with 256 threads that keep four steps and load the others again, 9.6; with 1024: 11)
    if (PX * NCH > 256) launch(input_fill_kernel<512, 3>, 512);
    else launch(input_fill_kernel<256, 1>, 256);
    return hipGetLastError();
}

hipError_t launch_layout_convert(const float *src, int N, int C, int H, int W, int src_n4, float *dst,
                                 hipStream_t st)
{
    const long long CHW = (long long)C * H * W;
    const long long n = (long long)((N + 3) / 4) * CHW;
    hipLaunchKernelGGL(layout_convert_kernel, dim3(blocks_for(n, kBlock)), dim3(kBlock), 0, st, src, N,
                       CHW, src_n4, dst);
    return hipGetLastError();
}

hipError_t launch_maxpool2x2(const float *x, int N, int C, int H, int W, float *y, int n4,
                             hipStream_t st)
{
    const int Ho = H / 2, Wo = W / 2;
    if (n4) {
        const long long GC = (long long)((N + 3) / 4) * C;
        const long long m = GC * Ho * Wo;
        if (m == 0) return hipSuccess;
        hipLaunchKernelGGL(maxpool2x2_n4_kernel, dim3(blocks_for(m, kBlock)), dim3(kBlock), 0, st,
                           reinterpret_cast<const float4 *>(x), GC, H, W, Ho, Wo,
                           reinterpret_cast<float4 *>(y));
        return hipGetLastError();
    }
    const long long n = (long long)N * C * Ho * Wo;
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(maxpool2x2_kernel, dim3(blocks_for(n, kBlock)), dim3(kBlock), 0, st, x,
                       (long long)N * C, H, W, Ho, Wo, y);
    return hipGetLastError();
}

}  // namespace fscnn
