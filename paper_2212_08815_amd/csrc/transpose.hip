// Sparse matrix transpose (Alg. 3) and sparse 3-D tensor transpose O_whc -> O_chw (Alg. 4).
//
// Both reorder stored nodes: every node moves to a new row (its "bucket") and the nodes of a
// new row are ordered by a "key" that is unique inside the row:
//   matrix, rows -> columns:   bucket = column of the node,  key = its old row;
//   tensor, O_whc -> O_chw:    old row = c*H + h lists w;  bucket = w*H + h,  key = c.
// The paper does this with a sequential walk that advances one cursor per new row (the vector
// v of Alg. 3) - a stable counting sort.  The same result is computed here in passes whose
// outcome does not depend on thread order, with scratch of O(nodes + new rows):
//   1. count the nodes of every bucket (integer atomic adds: the sums are order-independent);
//   2. exclusive scan of the counts = the new pointer array;
//   3. drop every node into its bucket's segment of a scratch copy, at a position handed out by
//      an atomic cursor - the segment then holds the right nodes in an arbitrary order;
//   4. every node of the scratch copy counts the nodes of its segment with a smaller key - its
//      rank, since keys are unique inside a bucket - and lands at pointer[bucket] + rank.
// The arbitrary order of step 3 never reaches the result.  Step 4 costs the sum of the squared
// bucket sizes.  Integer work only; values are copied bit for bit.
//
// Those passes take up to 8 launches, binary searches over the row pointers per node, global atomics and
// the rank's loop: at 28 x 28 x 512 with 31 % stored (124 000 nodes, 2.1 MB moved) 83 us, of them 27 + 29
// in counting and dropping, 21 in ranking.  Where the scratch allows (use_tiles below) three launches over
// tiles of the dense shape do it in 15, now the host call (112 x 112 x 512, 50 % stored: 693 -> 51, of 73 while a
// lane's nodes were loaded after the row's ends, values after the indices, and again for the second walk;
// a 1024 x 8192 matrix, 30 %: 324 -> 75, bound by its 4-byte stores; 64 x 64, 10 %: 26 -> 15):
//   1. a work-group takes RG (up to 32) consecutive keys and a panel of up to kPanel buckets of one
//      plane (a matrix is one plane, a tensor has one per h).  Its nodes set bit (key mod RG) of the
//      bucket's word in LDS; the number of bits is the tile's count for the bucket;
//   2. per bucket, the counts of the key groups become offsets inside the bucket, and the bucket
//      totals are scanned per block of 256 buckets;
//   3. the tile's words are built again and every node lands at (start of the bucket) + (offset of
//      its key group) + (number of set bits below its own).
#include <mutex>

#include "internal.h"

namespace fscnn {

namespace {

constexpr int kBlock = 256;

__global__ void __launch_bounds__(kBlock) reorder_clear_kernel(uint32_t *__restrict__ p, long long n)
{
    const long long i = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// Row of entry e: the last r with rowptr[r] <= e (rows may be empty).
__device__ inline int row_of(const int *__restrict__ rowptr, int n_rows, long long e)
{
    int lo = 0, hi = n_rows;  // invariant: rowptr[lo] <= e < rowptr[hi]
    while (hi - lo > 1) {
        const int mid = lo + (hi - lo) / 2;
        if (rowptr[mid] <= e) lo = mid; else hi = mid;
    }
    return lo;
}

struct Dest {
    long long bucket;
    int key;
    bool ok;
};

// TENSOR = false: n_cols columns;  TENSOR = true: n_cols = W, H rows per channel.
template <bool TENSOR>
__device__ inline Dest dest_of(int row, uint32_t col, int n_cols, int H)
{
    Dest d;
    d.ok = col < (uint32_t)n_cols;  // a corrupt index is dropped, never followed
    if (TENSOR) {
        const int c = row / H, h = row - c * H;
        d.bucket = (long long)col * H + h;
        d.key = c;
    } else {
        d.bucket = col;
        d.key = row;
    }
    return d;
}

template <bool TENSOR>
__global__ void __launch_bounds__(kBlock) reorder_count_kernel(const int *__restrict__ rowptr,
                                                               const uint32_t *__restrict__ idx,
                                                               int n_rows, int n_cols, int H,
                                                               long long nnz, int *__restrict__ cnt)
{
    const long long e = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (e >= nnz) return;
    const Dest d = dest_of<TENSOR>(row_of(rowptr, n_rows, e), idx[e], n_cols, H);
    if (d.ok) atomicAdd(&cnt[d.bucket], 1);
}

// cursor[b] = tptr[b]: where the next node of bucket b is dropped
__global__ void __launch_bounds__(kBlock) reorder_cursor_kernel(const int *__restrict__ tptr,
                                                                long long n_buckets, int *__restrict__ cursor)
{
    const long long b = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (b < n_buckets) cursor[b] = tptr[b];
}

template <bool TENSOR>
__global__ void __launch_bounds__(kBlock) reorder_drop_kernel(
    const int *__restrict__ rowptr, const uint32_t *__restrict__ idx, const float *__restrict__ val,
    int n_rows, int n_cols, int H, long long nnz, int *__restrict__ cursor,
    uint32_t *__restrict__ skey, float *__restrict__ sval)
{
    const long long e = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (e >= nnz) return;
    const Dest d = dest_of<TENSOR>(row_of(rowptr, n_rows, e), idx[e], n_cols, H);
    if (!d.ok) return;
    const int p = atomicAdd(&cursor[d.bucket], 1);
    if (p < nnz) {
        skey[p] = (uint32_t)d.key;
        sval[p] = val[e];
    }
}

// One thread per position of the scratch copy: its bucket is the segment of tptr that holds the
// position; its rank is the number of smaller keys in that segment.
__global__ void __launch_bounds__(kBlock) reorder_place_kernel(const int *__restrict__ tptr,
                                                               long long n_buckets, long long total,
                                                               const uint32_t *__restrict__ skey,
                                                               const float *__restrict__ sval,
                                                               uint32_t *__restrict__ tidx,
                                                               float *__restrict__ tval)
{
    const long long p = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (p >= total || p >= tptr[n_buckets]) return;   // past the last node that was kept
    // last b with tptr[b] <= p (buckets may be empty)
    long long lo = 0, hi = n_buckets;
    while (hi - lo > 1) {
        const long long mid = lo + (hi - lo) / 2;
        if (tptr[mid] <= p) lo = mid; else hi = mid;
    }
    const int a = tptr[lo], b = tptr[lo + 1];
    const uint32_t key = skey[p];
    int rank = 0;
    for (int q = a; q < b; ++q) rank += skey[q] < key ? 1 : 0;
    tidx[a + rank] = key;
    tval[a + rank] = sval[p];
}

// ---- the tiled form
constexpr int kPanel = 4096;        // buckets of a tile at most: 16 KB of words, 16 KB of starts
constexpr int kMaxSums = 256;       // blocks of 256 buckets whose totals step 3 scans by itself

// Nodes of a row that a lane has in flight or in registers: four, LPR apart, from entry e on.  With `values` their values too
// (where a tile sees the whole row: of several panels each would load them for a few nodes).
struct Nodes {
    int e, hi;                          // hi: end of the row
    uint32_t w[4];
    float v[4];
};
__device__ inline Nodes load_nodes(const uint32_t *__restrict__ idx, const float *__restrict__ val, bool values, int e, int hi, int LPR)
{
    Nodes n;
    n.e = e;
    n.hi = hi;
#pragma unroll
    for (int u = 0; u < 4; ++u) n.w[u] = hi - e > u * LPR ? idx[e + u * LPR] : 0xffffffffu;
#pragma unroll
    for (int u = 0; u < 4; ++u) n.v[u] = values && hi - e > u * LPR ? val[e + u * LPR] : 0.0f;
    return n;
}
// Lane's first entry and the end of row `key` of plane h; nothing past the last key.
__device__ inline int2 row_span(const int *__restrict__ rowptr, int H, int C, int h, int key, bool mine, int LPR, int nnz)
{
    if (!mine || key >= C) return make_int2(0, 0);
    const int lo = rowptr[key * H + h], hi = rowptr[key * H + h + 1];
    return make_int2((lo < 0 ? 0 : lo) + (int)threadIdx.x % LPR, hi > nnz ? nnz : hi);
}
__device__ inline Nodes first_nodes(const int *__restrict__ rowptr, const uint32_t *__restrict__ idx, const float *__restrict__ val,
                                    bool values, int H, int C, int h, int c0, int RG, int LPR, int nnz)
{
    const int r = (int)threadIdx.x / LPR;
    const int2 s = row_span(rowptr, H, C, h, c0 + r, r < RG, LPR, nnz);
    return load_nodes(idx, val, values, s.x, s.y, LPR);
}

// f(key mod RG, bucket of the plane relative to the panel, entry, its value if loaded) for every node of the tile.
// LPR lanes share a row (use_tiles says how many).  `n`: the lane's first nodes, which a caller that walks
// twice loads once; a row's ends are loaded while the row before is worked on.
template <class Fn>
__device__ inline void for_tile_nodes(Nodes n, const int *__restrict__ rowptr, const uint32_t *__restrict__ idx,
                                      const float *__restrict__ val, bool values, int H, int C, int h, int c0, int RG, int w0, int wn,
                                      int LPR, int nnz, Fn f)
{
    const int step = kBlock / LPR;
    for (int r = (int)threadIdx.x / LPR; r < RG && c0 + r < C; r += step) {
        const int2 next = row_span(rowptr, H, C, h, c0 + r + step, r + step < RG, LPR, nnz);
        for (;;) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t q = n.w[u] - (uint32_t)w0;   // (an index outside the panel, or corrupt, wraps past it)
                if (n.hi - n.e > u * LPR && q < (uint32_t)wn) f(r, (int)q, n.e + u * LPR, n.v[u]);
            }
            if (n.hi - n.e <= 4 * LPR) break;
            n = load_nodes(idx, val, values, n.e + 4 * LPR, n.hi, LPR);
        }
        n = load_nodes(idx, val, values, next.x, next.y, LPR);
    }
}

struct Tile {
    int h, g, w0, wn;
};
__device__ inline Tile tile_of(int n_cols, int H, int panels, int pw)
{
    Tile t;
    const int b = blockIdx.x;
    t.w0 = (b % panels) * pw;
    t.wn = n_cols - t.w0 < pw ? n_cols - t.w0 : pw;
    t.h = (b / panels) % H;
    t.g = b / panels / H;
    return t;
}

// cnt[g * n_buckets + bucket], bucket = w * H + h
__global__ void __launch_bounds__(kBlock) tile_count_kernel(const int *__restrict__ rowptr,
                                                            const uint32_t *__restrict__ idx, int n_cols, int H, int C,
                                                            int RG, int panels, int pw, int LPR, int nnz,
                                                            long long n_buckets, unsigned short *__restrict__ cnt)
{
    extern __shared__ uint32_t word[];
    const Tile t = tile_of(n_cols, H, panels, pw);
    const Nodes first = first_nodes(rowptr, idx, nullptr, false, H, C, t.h, t.g * RG, RG, LPR, nnz);
    for (int w = threadIdx.x; w < t.wn; w += kBlock) word[w] = 0u;
    __syncthreads();
    for_tile_nodes(first, rowptr, idx, nullptr, false, H, C, t.h, t.g * RG, RG, t.w0, t.wn, LPR, nnz,
                   [&](int r, int w, int, float) { atomicOr(&word[w], 1u << r); });
    __syncthreads();
    for (int w = threadIdx.x; w < t.wn; w += kBlock)
        cnt[t.g * n_buckets + (long long)(t.w0 + w) * H + t.h] = (unsigned short)__popc(word[w]);
}

// cnt -> offsets of the groups inside their bucket (in place); first[b] = start of bucket b inside its
// block of 256 buckets; sums[block] = nodes of the block.  kParts threads share a bucket, each a run of
// its groups: it adds them up, then writes their offsets; 16 loads in flight, read once where there are no
// more (one thread per bucket took longer than the rest of the transpose where keys are many and buckets few).
constexpr int kParts = 4;
__global__ void __launch_bounds__(kBlock *kParts) tile_offsets_kernel(unsigned short *__restrict__ cnt, int n_buckets,
                                                                      int G, int *__restrict__ first,
                                                                      int *__restrict__ sums)
{
    __shared__ int part_sum[kParts][kBlock], wave_sum[kBlock / 64];
    const int t = threadIdx.x % kBlock, part = threadIdx.x / kBlock;
    const int b = blockIdx.x * kBlock + t, lane = threadIdx.x & 63, wave = t >> 6;
    const int per = (G + kParts - 1) / kParts;
    const int ga = part * per, gb = b < n_buckets ? (ga + per < G ? ga + per : G) : 0;
    unsigned short *p = cnt + b;
    int v[16];                             // the last 16 that were read
    auto read = [&](int g0) {
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = g0 + u < gb ? p[(long long)(g0 + u) * n_buckets] : 0;
    };
    int sum = 0;
    for (int g0 = ga; g0 < gb; g0 += 16) {
        read(g0);
#pragma unroll
        for (int u = 0; u < 16; ++u) sum += v[u];
    }
    part_sum[part][t] = sum;
    __syncthreads();
    int base = 0, total = 0;
#pragma unroll
    for (int q = 0; q < kParts; ++q) {
        if (q < part) base += part_sum[q][t];
        total += part_sum[q][t];
    }
    for (int g0 = ga; g0 < gb; g0 += 16) {
        if (per > 16) read(g0);            // (else they are there)
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            if (g0 + u < gb) p[(long long)(g0 + u) * n_buckets] = (unsigned short)base;
            base += v[u];
        }
    }
    int incl = total;
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
    }
    if (part == 0 && lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int before = 0;
    for (int i = 0; i < wave; ++i) before += wave_sum[i];
    if (part == 0 && b < n_buckets) first[b] = before + incl - total;
    if (threadIdx.x == kBlock - 1) sums[blockIdx.x] = before + incl;
}

__global__ void __launch_bounds__(kBlock) tile_place_kernel(
    const int *__restrict__ rowptr, const uint32_t *__restrict__ idx, const float *__restrict__ val, int n_cols, int H,
    int C, int RG, int panels, int pw, int LPR, int nnz, long long n_buckets, const unsigned short *__restrict__ cnt,
    const int *__restrict__ first, const int *__restrict__ sums, int nsums, int *__restrict__ tptr,
    uint32_t *__restrict__ tidx, float *__restrict__ tval)
{
    extern __shared__ uint32_t word[];
    int *start = reinterpret_cast<int *>(word + pw);
    __shared__ int block_start[kMaxSums], wave_sum[kBlock / 64];
    const Tile t = tile_of(n_cols, H, panels, pw);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool values = panels == 1;
    const Nodes nodes = first_nodes(rowptr, idx, val, values, H, C, t.h, t.g * RG, RG, LPR, nnz);
    for (int w = threadIdx.x; w < t.wn; w += kBlock) word[w] = 0u;
    // starts of the blocks of buckets (kMaxSums == kBlock: one each)
    const int mine = (int)threadIdx.x < nsums ? sums[threadIdx.x] : 0;
    int incl = mine;
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int before = 0;
    for (int i = 0; i < wave; ++i) before += wave_sum[i];
    block_start[threadIdx.x] = before + incl - mine;
    if (blockIdx.x == 0 && threadIdx.x == kBlock - 1) tptr[n_buckets] = before + incl;
    for_tile_nodes(nodes, rowptr, idx, val, false, H, C, t.h, t.g * RG, RG, t.w0, t.wn, LPR, nnz,
                   [&](int r, int w, int, float) { atomicOr(&word[w], 1u << r); });
    __syncthreads();
    for (int w = threadIdx.x; w < t.wn; w += kBlock) {
        const int b = (t.w0 + w) * H + t.h;
        const int at = block_start[b / kBlock] + first[b];
        if (t.g == 0) tptr[b] = at;
        start[w] = at + cnt[t.g * n_buckets + b];
    }
    __syncthreads();
    for_tile_nodes(nodes, rowptr, idx, val, values, H, C, t.h, t.g * RG, RG, t.w0, t.wn, LPR, nnz, [&](int r, int w, int e, float v) {
        const int p = start[w] + __popc(word[w] & ((1u << r) - 1u));
        if (p < nnz) {   // (holds for every node of a valid pointer array)
            tidx[p] = (uint32_t)(t.g * RG + r);
            tval[p] = values ? v : val[e];
        }
    });
}
static_assert(kMaxSums == kBlock, "step 3 scans one sum per thread");

inline unsigned blocks_for(long long n) { return (unsigned)((n + kBlock - 1) / kBlock); }

// scratch layout (32-bit words): cnt[n_buckets] | scan scratch | cursor[n_buckets] | skey[nnz] | sval[nnz]
struct Layout {
    long long cnt, scan, cursor, skey, sval, words;
};
inline Layout layout_of(long long n_buckets, long long nnz)
{
    Layout l;
    l.cnt = 0;
    l.scan = n_buckets;
    l.cursor = l.scan + scan_tmp_elems(n_buckets);
    l.skey = l.cursor + n_buckets;
    l.sval = l.skey + nnz;
    l.words = l.sval + nnz;
    return l;
}

// How the tiled form would run.  Scratch, in 32-bit words: first[n_buckets] | sums[nsums] | cnt (16 bits each)
struct TilePlan {
    bool ok;
    int RG, G, panels, pw, LPR, nsums;
    long long blocks;
};
// The tiled form wants its counts (16 bits per bucket and key group) in the scratch that the callers bring
// for the node-by-node form, which ties it to about 1 % stored nodes and more; step 3 scans at most 256
// block totals (65536 buckets); a bucket's offsets fit 16 bits below 65536 keys.  As many keys per tile as
// still give a work-group for every CU or leave it few nodes (more groups are more counts), 8 at least
// (1024 x 64, 10 %: 37 us with 128 groups of 8, 15 with 32 of 32).
TilePlan use_tiles(int n_cols, int H, int C, long long n_buckets, long long nnz)
{
    TilePlan t{};
    t.nsums = (int)((n_buckets + kBlock - 1) / kBlock);
    if (t.nsums > kMaxSums || C > 65535 || nnz <= 0) return t;
    t.panels = (n_cols + kPanel - 1) / kPanel;
    t.pw = (n_cols + t.panels - 1) / t.panels;
    const long long room = layout_of(n_buckets, nnz).words;
    for (int rg = 32; rg >= 8; rg /= 2) {
        const long long G = (C + rg - 1) / rg, blocks = G * H * t.panels;
        if (n_buckets + t.nsums + (G * n_buckets + 1) / 2 > room || blocks * kBlock > 0xffffffffLL) break;
        if (blocks > 1024 && nnz < 16 * blocks) break;   // nearly empty tiles, each with its fixed part
        t.ok = true;
        t.RG = rg;
        t.G = (int)G;
        t.blocks = blocks;
        if (blocks >= 256 || nnz <= 512 * blocks) break;
    }
    // Lanes per row: each has four nodes in flight, so a third of a row's average takes most rows in one go; more where a
    // tile has fewer rows than that makes room for.
    const long long avg = nnz / ((long long)C * H);
    t.LPR = 4;
    while (t.LPR < 64 && (3 * t.LPR < avg || t.LPR * t.RG < kBlock)) t.LPR *= 2;
    return t;
}

// Scratch of the entry point that allocates nothing: one copy per GPU, held until the process
// ends.  Host code never passes this name to a kernel: it is a host-side stand-in, the device
// address comes from hipGetSymbolAddress (static_scratch below).
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
void *scratch_ptr[kMaxDevices];   // device address of `scratch` on each GPU, once looked up

}  // namespace

hipError_t static_scratch(void **ptr)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));   // with `dev` current: this GPU's copy
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        scratch_ptr[dev] = p;
    }
    *ptr = scratch_ptr[dev];
    return hipSuccess;
}

long long reorder_workspace_bytes(long long n_buckets, long long nnz)
{
    if (n_buckets <= 0 || nnz < 0 || n_buckets >= (1LL << 31) || nnz >= (1LL << 31)) return -1;
    return 4 * layout_of(n_buckets, nnz).words;
}

hipError_t launch_reorder(bool tensor, const int *rowptr, const uint32_t *idx, const float *val,
                          int n_rows, int n_cols, int H, long long n_buckets, long long nnz,
                          int *tptr, uint32_t *tidx, float *tval, void *workspace, hipStream_t st)
{
    int *ws = static_cast<int *>(workspace);
    const int C = n_rows / H;   // keys (a matrix is one plane, H = 1)
    const TilePlan tp = use_tiles(n_cols, H, C, n_buckets, nnz);
    if (tp.ok) {
        int *first = ws, *sums = ws + n_buckets;
        unsigned short *groups = reinterpret_cast<unsigned short *>(sums + tp.nsums);
        hipLaunchKernelGGL(tile_count_kernel, dim3((unsigned)tp.blocks), dim3(kBlock), tp.pw * 4, st, rowptr, idx,
                           n_cols, H, C, tp.RG, tp.panels, tp.pw, tp.LPR, (int)nnz, n_buckets, groups);
        hipLaunchKernelGGL(tile_offsets_kernel, dim3((unsigned)tp.nsums), dim3(kBlock * kParts), 0, st, groups, (int)n_buckets,
                           tp.G, first, sums);
        hipLaunchKernelGGL(tile_place_kernel, dim3((unsigned)tp.blocks), dim3(kBlock), tp.pw * 8, st, rowptr, idx, val,
                           n_cols, H, C, tp.RG, tp.panels, tp.pw, tp.LPR, (int)nnz, n_buckets, groups, first, sums,
                           tp.nsums, tptr, tidx, tval);
        return hipGetLastError();
    }
    const Layout l = layout_of(n_buckets, nnz);
    int *cnt = ws + l.cnt, *cursor = ws + l.cursor;
    uint32_t *skey = reinterpret_cast<uint32_t *>(ws + l.skey);
    float *sval = reinterpret_cast<float *>(ws + l.sval);
    hipLaunchKernelGGL(reorder_clear_kernel, dim3(blocks_for(n_buckets)), dim3(kBlock), 0, st,
                       reinterpret_cast<uint32_t *>(cnt), n_buckets);
    if (nnz > 0) {
        if (tensor)
            hipLaunchKernelGGL(reorder_count_kernel<true>, dim3(blocks_for(nnz)), dim3(kBlock), 0, st,
                               rowptr, idx, n_rows, n_cols, H, nnz, cnt);
        else
            hipLaunchKernelGGL(reorder_count_kernel<false>, dim3(blocks_for(nnz)), dim3(kBlock), 0, st,
                               rowptr, idx, n_rows, n_cols, H, nnz, cnt);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = launch_exclusive_scan(cnt, tptr, n_buckets, ws + l.scan, nullptr, false, st);
    if (e != hipSuccess || nnz == 0) return e;
    hipLaunchKernelGGL(reorder_cursor_kernel, dim3(blocks_for(n_buckets)), dim3(kBlock), 0, st, tptr,
                       n_buckets, cursor);
    if (tensor)
        hipLaunchKernelGGL(reorder_drop_kernel<true>, dim3(blocks_for(nnz)), dim3(kBlock), 0, st, rowptr,
                           idx, val, n_rows, n_cols, H, nnz, cursor, skey, sval);
    else
        hipLaunchKernelGGL(reorder_drop_kernel<false>, dim3(blocks_for(nnz)), dim3(kBlock), 0, st, rowptr,
                           idx, val, n_rows, n_cols, H, nnz, cursor, skey, sval);
    // nodes with a corrupt index were skipped: the kernel reads the number of kept nodes from the
    // pointer array's last element and places no position beyond it
    hipLaunchKernelGGL(reorder_place_kernel, dim3(blocks_for(nnz)), dim3(kBlock), 0, st, tptr, n_buckets,
                       nnz, skey, sval, tidx, tval);
    return hipGetLastError();
}

}  // namespace fscnn
