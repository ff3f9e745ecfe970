// 1x1 filters at stride 1 without padding: y = W x, W sparse (a row per output channel), x dense with a column per pixel.
//
// The tiled kernels (conv_sf.hip) stage every input channel for each group of 64 output channels, whether or not a filter stores
// an entry there; with 3 to 50 entries a filter that, its barriers and the latency of a chain of chunks is what a layer takes.  Here nothing is
// staged.  A wave owns 256 adjacent pixels (four a lane; with N4 tensors pixel x image) and takes output channels one after the other: an entry is
// one 16-byte load a lane from its channel's plane and four multiply-adds, the entries' channels and values come through scalar
// loads, eight at a time, so that eight loads are in flight.  Four partial sums per output, added at the end: shorter chains of roundings
// than one sum in the order of the entries.  Work-groups of one pixel block run next to each other on one XCD and find its planes in the L2.
// What bounds it: few images, two round trips to memory behind a launch; many, the 64 bytes a clock that a CU takes from its
// L1 (4 bytes per multiply-add; 35 of them reached by 512 -> 256 at 26x26, N = 8, 5 % stored, N4, 11.2 us) or the tensors' way from and to
// memory (225 -> 741 at 79x146, N = 9, 1 %, N4: 535 MB in 221 us, 17 bytes a clock from the L1).  Nothing is kept for it: no plan.
// 5 % stored, us before (contracted in fp32 or gathered) and so: 256 -> 128 at 44x44, N = 1: 11.4, 5.4; 1024 -> 512 at 11x11, N = 1: 20.2, 6.7;
// 512 -> 256 at 8x8, N = 18, 16 % stored, N4: 17.9, 10.8; 225 -> 741 at 79x146, N = 9, 1 %, N4: 471, 236.  At 52x52 and N = 32 the planes' way
// through the L1 makes it the slower one (256 -> 128: 33 gathered, 60): pointwise() in api.hip draws the line.
#include <type_traits>

#include "internal.h"
#include "lds_dma.h"

namespace fscnn {

namespace {

struct PwArgs {
    const float *x;
    float *y;
    const float *bias;
    const int *rowptr;
    const uint32_t *idx;
    const float *val;
    int C, HW, K, act, rows, nrg, pxb, nblk;   // HW: pixels x images of a group; rows: per wave; row groups; pixel blocks of a group of images
};

constexpr int kPwWaves = 4, kPwPixels = 256;

__device__ inline int xcd_neighbours(int bid, int nblk)   // (as the tiled kernels do: consecutive ids on one XCD)
{
    const int q = nblk >> 3, rem = nblk & 7, xcd = bid & 7, slot = bid >> 3;
    return xcd < rem ? xcd * (q + 1) + slot : rem * (q + 1) + (xcd - rem) * q + slot;
}

__global__ void __launch_bounds__(kPwWaves * 64) pointwise_kernel(const PwArgs a)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lid = xcd_neighbours(blockIdx.x, a.nblk);
    const int rg = lid % a.nrg, pb = lid / a.nrg, g = pb / a.pxb;
    // (the last lane with pixels overlaps the one before it: all its four lie in the plane)
    const int p = (pb % a.pxb) * kPwPixels + lane * 4, px = p + 4 <= a.HW ? p : a.HW - 4;
    const bool live = p < a.HW;
    const int bytes = a.HW * 4;
    // (the launch checked that a group's channels lie within 2^31 bytes)
    const __amdgpu_buffer_rsrc_t xs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.x + (long long)g * a.C * a.HW), 0, a.C * bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t ys = __builtin_amdgcn_make_buffer_rsrc(a.y + (long long)g * a.K * a.HW, 0, a.K * bytes, 0x00020000);
    const int off = live ? px * 4 : (int)0x80000000;
    typedef unsigned int u4v __attribute__((ext_vector_type(4)));
    const int k0 = (rg * kPwWaves + wave) * a.rows, k1 = k0 + a.rows < a.K ? k0 + a.rows : a.K;
    for (int k = k0; k < k1; ++k) {
        const int lo = a.rowptr[k], hi = a.rowptr[k + 1];
        f4v acc[4] = {};
        auto plane = [&](uint32_t c) { return __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(xs, off, (int)c * bytes, 0)); };
        int i = lo;
        if (i + 8 <= hi) {
            uint32_t c[8];
            float w[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) { c[u] = a.idx[i + u]; w[u] = a.val[i + u]; }
            for (;;) {
                f4v v[8];
                float m[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) { v[u] = plane(c[u]); m[u] = w[u]; }
                i += 8;
                const bool more = i + 8 <= hi;
                if (more) {                           // the next entries, while the planes are on their way
#pragma unroll
                    for (int u = 0; u < 8; ++u) { c[u] = a.idx[i + u]; w[u] = a.val[i + u]; }
                }
#pragma unroll
                for (int u = 0; u < 8; ++u)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[u % 4][e] = __builtin_fmaf(m[u], v[u][e], acc[u % 4][e]);
                if (!more) break;
            }
        }
        auto take = [&](auto count) {                 // the rest, in one chain: a filter of few entries has no more roundings than they are
            constexpr int n = decltype(count)::value;
            float w[n];
            f4v v[n];
#pragma unroll
            for (int u = 0; u < n; ++u) { v[u] = plane(a.idx[i + u]); w[u] = a.val[i + u]; }
#pragma unroll
            for (int u = 0; u < n; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[0][e] = __builtin_fmaf(w[u], v[u][e], acc[0][e]);
            i += n;
        };
        if ((hi - i) & 4) take(std::integral_constant<int, 4>{});
        if ((hi - i) & 2) take(std::integral_constant<int, 2>{});
        if ((hi - i) & 1) take(std::integral_constant<int, 1>{});
        f4v s = (acc[0] + acc[1]) + (acc[2] + acc[3]);
        const float b = a.bias ? a.bias[k] : 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = act_apply(s[e] + b, a.act);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4v, s), ys, off, k * bytes, 0);
    }
}

}  // namespace

static int pw_rows(long long blocks, int K)
{
    // as many rows a wave as leave 16 waves a CU: the pixels' planes are shared by the rows of a wave through the L1
    int rows = 1;
    while (rows < 8 && blocks * ((K + kPwWaves * 2 * rows - 1) / (kPwWaves * 2 * rows)) * kPwWaves >= 4096) rows *= 2;
    return rows;
}

bool pointwise_serves(int N, int C, int H, int W, int K, bool n4)
{
    const long long HW = (long long)H * W * (n4 ? 4 : 1), G = n4 ? (N + 3) / 4 : N;
    const long long most = 0x7ffffff0LL, blocks = (HW + kPwPixels - 1) / kPwPixels * G;
    return HW >= 4 && HW * C * 4 < most && HW * K * 4 < most && blocks * ((K + kPwWaves - 1) / kPwWaves) * 256 <= 0xffffffffLL;
}

double pointwise_us(int N, int C, int H, int W, int K, bool n4, long long nnz)
{
    // a launch, the tensors' way from memory (channels without an entry are not read), the planes' way to the CUs, the entries' latency: over 130 layers
    // within 23 % (standard deviation), the choice by it 1 % slower than the faster of the two on average
    const double px = (double)H * W * (n4 ? (N + 3) / 4 * 4 : N), read = 0.8 * (nnz < C ? (double)nnz : C);
    return 4.5 + 4.0 * px * (read + K) / 4.8e6 + 4.0 * px * nnz / 25e6 + 0.06 * nnz / K;
}

hipError_t launch_pointwise(const int *rowptr, const uint32_t *idx, const float *val, const float *x, int N, int C, int H, int W, int K,
                            bool n4, const float *bias, int act, float *y, hipStream_t st)
{
    if (!pointwise_serves(N, C, H, W, K, n4)) return hipErrorInvalidValue;
    PwArgs a = {x, y, bias, rowptr, idx, val, C, H * W * (n4 ? 4 : 1), K, act, 0, 0, 0, 0};
    a.pxb = (a.HW + kPwPixels - 1) / kPwPixels;
    const long long blocks = (long long)a.pxb * (n4 ? (N + 3) / 4 : N);
    a.rows = pw_rows(blocks, K);
    a.nrg = (K + kPwWaves * a.rows - 1) / (kPwWaves * a.rows);
    const long long nblk = blocks * a.nrg;
    if (nblk <= 0 || nblk * (kPwWaves * 64) > 0xffffffffLL) return hipErrorInvalidValue;
    a.nblk = (int)nblk;
    hipLaunchKernelGGL(pointwise_kernel, dim3((unsigned)nblk), dim3(kPwWaves * 64), 0, st, a);
    return hipGetLastError();
}

}  // namespace fscnn
