// Convolution as a dense contraction on the matrix cores (fp32 MFMA), for the calls whose operand
// is too dense for a gather of single multiply-adds to pay, and which the contraction in bfloat16 parts
// (contract_split.hip: 3x3 and 5x5) does not serve or is not estimated to serve a tenth faster:
//   * a compressed filter bank that stores a large share of its entries (or whose extent no gather
//     configuration serves) applied to a dense NCHW tensor;
//   * a compressed activation (per-pixel channel lists) with a dense filter bank.
// The gather kernels run one LDS word per multiply-add on the vector ALUs (about 55 TFLOP/s of
// stored weights at best); v_mfma_f32_16x16x4_f32 multiplies and adds in fp32 at 256 flop per clock
// and CU whatever the operands hold (154 TFLOP/s for a large fp32 matrix product on this chip), so
// with a share d of non-zeros the contraction wins from d of about a third of that rate ratio on.
//
// How it is mapped:
//   * y[k, p] = sum over (c, r, s) of w[k, c, r, s] * x[c, p shifted by (r, s)]: output channels are
//     the rows of the matrix product, output pixels its columns.  A work-group owns 16*MW channels
//     and T = 16*NT pixels; MW waves lie along the channels (16 rows each), and KS slices of waves
//     divide every chunk of 16*KS input channels among them, so that small problems keep enough
//     waves in flight; the slices' sums are added through LDS, in order, at the end.
//   * pixels are numbered across rows and images (inside a panel of SW columns for wide images), so
//     a tile need not be a rectangle: 28x28 images waste nothing in tiles of 112 or 208 pixels.
//     The tile's input rows (with halo) form a stripe of "virtual rows", an image contributing
//     (Ho-1)*stride + R of them, out-of-image ones being zero.
//   * LDS holds the stripe with four channels interleaved per pixel: one ds_read_b128 per (tap, 16
//     pixels) gives a lane the B operands of four MFMAs (lane group q = lane/16 owns channels 4q..4q+3
//     of the slice's 16).  Two buffers; the loads of the next chunk are in flight while a chunk is
//     multiplied, and are written to LDS half way through.
//   * the A operands go from global memory to registers, a chunk ahead.  A packed bank holds them
//     as the lanes want them, [16 rows][16 channels][tap][lane][4]: one 16-byte load, 1 KB per wave
//     and tap.  (Read as [c][tap][k] with a power of two of rows, every load of a work-group fell on
//     the same two of an L2's sixteen channels.)  A lane of a K x C x 3 x 3 bank needs 36 consecutive
//     floats a chunk, nine 16-byte loads.
// What bounds it: the matrix unit on full tiles (measured where the parts serve now: 512 -> 512 at 28x28, N = 8: 253 us back to
// back, the unit busy 78 % of the clocks from a dense tensor, 69 to 72 from lists; the LDS 20 %, waves waiting 16 to 20 % of
// their time); where a launch is a round of short work-groups (96 -> 256 5x5 at 27x27, N = 8: busy 54 %) its loads and stores as well.
//
// Non-finite operands: a gather never multiplies an entry that is not stored, so 0 * Inf cannot
// appear there.  Dense tensors are checked while they are staged (a stripe that holds an Inf or NaN
// makes the work-group recompute its tile the slow way, walking the stored entries); filter banks
// that meet compressed activations likewise, and those of calls that the direct kernel would serve: it
// skips the entries that fall outside the image, which meet staged zeros here.
#include <type_traits>

#include "internal.h"
#include "lds_dma.h"

namespace fscnn {

namespace {

enum { kSrcDense = 0, kSrcLists = 1 };   // where x comes from
enum { kWKC = 0, kWPacked = 1 };         // weights as K x C x R x S, or packed in the order of the A operands

// 64-pixel rounds of the staging loop, which bounds a tile's stripe: their registers are per lane
constexpr int it_max(int KS) { return KS >= 4 ? 4 : 8; }
constexpr int kLdsMax = 160 * 1024 - 512;
constexpr int kOut = 0x7ffffff0;         // beyond any descriptor's range: the buffer load returns 0

struct DcArgs {
    const float *x;                      // dense source
    const int *cptr;                     // list source
    const uint32_t *cidx;
    const float *xval;
    const int *gate;                     // lists: if not NULL, another kernel serves the call unless gate_from <= *gate < gate_to
    int gate_from, gate_to;
    const float *w;
    const int *wflag;                    // kWPacked: non-zero if the bank holds an Inf or NaN; NULL: it does not matter
    const int *rowptr;                   // dense source: the stored entries, for the slow way
    const uint32_t *idx;
    const float *val;
    const float *bias;
    float *y;
    int N, C, H, W, K, nslice, R, S, Ho, Wo, sh, sw, ph, pw, act, NCP;
    int SW, tpp, pitch, PL, VR, NKT, buf_bytes;
    uint32_t m_pitch, m_vr, m_sw, m_ho;  // reciprocals for div_by()
};

// x / d for a divisor whose reciprocal ceil(2^31 / d) the host computed; exact while x * d < 2^31
__device__ inline int div_by(int x, uint32_t m) { return (int)__umulhi((uint32_t)x * 2u, m); }
inline uint32_t recip_of(int d) { return (uint32_t)(((1LL << 31) + d - 1) / d); }

template <int MW_, int KS_, int NT_, int SRC_, int WSRC_, int RS_>
struct DcCfg {
    static constexpr int MW = MW_, KS = KS_, NT = NT_, SRC = SRC_, WSRC = WSRC_;
    static constexpr int RS = RS_;               // 9: 3x3, all of a chunk's A operands in registers; 0: any extent
    static constexpr int WAVES = MW * KS, NTH = WAVES * 64;
    static constexpr int IT = it_max(KS);
    static constexpr int CC = 16 * KS;           // input channels per chunk
    static constexpr int T = 16 * NT;            // pixels per work-group
    static constexpr int PPW = 4 / MW;           // planes of four channels a wave stages
    static constexpr int WPS = MW / 2;           // waves that share one 8-channel step of the lists
    static_assert(MW == 2 || MW == 4, "waves along the channels");
    static_assert(WAVES <= 16, "work-group size");
    // (one work-group of 8 waves per CU may use 256 registers a lane, of 16 waves 128)
    static constexpr int WPE = WAVES >= 16 ? 4 : 2;
    static constexpr int RED_BYTES = (KS - 1) * MW * 64 * NT * 16;
};

typedef uint32_t u4v __attribute__((ext_vector_type(4)));

// running maximum of magnitudes: at or above the bit pattern of infinity once an Inf or NaN was seen
__device__ inline void see(uint32_t &top, float v)
{
    const uint32_t b = __float_as_uint(v) & 0x7fffffffu;
    top = b > top ? b : top;
}

// one output the slow way: only stored entries are multiplied
template <class G> __device__ float slow_output(const DcArgs &a, int n, int k, int oy, int ox)
{
    const int RS = a.R * a.S;
    float acc = 0.0f;
    if constexpr (G::SRC == kSrcDense) {
        const float *xn = a.x + (long long)n * a.C * a.H * a.W;
        for (int i = a.rowptr[k]; i < a.rowptr[k + 1]; ++i) {
            const uint32_t f = a.idx[i];
            const int c = (int)(f / RS), rs = (int)(f % RS);
            const int iy = oy * a.sh - a.ph + rs / a.S, ix = ox * a.sw - a.pw + rs % a.S;
            if (iy >= 0 && iy < a.H && ix >= 0 && ix < a.W)
                acc = __builtin_fmaf(a.val[i], xn[((long long)c * a.H + iy) * a.W + ix], acc);
        }
    } else {
        for (int rs = 0; rs < RS; ++rs) {
            const int iy = oy * a.sh - a.ph + rs / a.S, ix = ox * a.sw - a.pw + rs % a.S;
            if (iy < 0 || iy >= a.H || ix < 0 || ix >= a.W) continue;
            const long long pix = ((long long)n * a.H + iy) * a.W + ix;
            for (int i = a.cptr[pix * a.NCP]; i < a.cptr[(pix + 1) * a.NCP]; ++i) {
                const long long c = a.cidx[i];
                const float wv = G::WSRC == kWKC ? a.w[((long long)k * a.C + c) * RS + rs]
                                                 : a.w[contract_packed_index(k, (int)c, rs, RS, a.nslice)];
                acc = __builtin_fmaf(a.xval[i], wv, acc);
            }
        }
    }
    return acc;
}

template <int I, int N, class F> __device__ inline void static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

template <class G>
__global__ void __launch_bounds__(G::NTH, G::WPE) contract_kernel(const DcArgs a)
{
    extern __shared__ __align__(256) char ldsb[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int mw = wave % G::MW, ks = wave / G::MW;
    const int j = lane & 15, q = lane >> 4;
    const int kt = blockIdx.x % a.NKT, tile = blockIdx.x / a.NKT;
    const int pan = tile / a.tpp;
    const int p0 = (tile % a.tpp) * G::T;
    const int ptot = a.N * a.Ho * a.SW;               // pixels of a panel
    const int plast = p0 + G::T < ptot ? p0 + G::T - 1 : ptot - 1;
    const int HW = a.H * a.W;
    auto virt = [&](int v) { return (v / a.Ho) * a.VR + (v % a.Ho) * a.sh; };   // first input row of output row v
    const int v0 = p0 / a.SW;
    const int u0 = virt(v0), nrow = virt(plast / a.SW) + a.R - u0;
    const int npx = nrow * a.pitch;
    const int n0 = v0 / a.Ho;

    // (here, where the arguments have arrived: at the top it cost every call one more round trip for them)
    if constexpr (G::SRC == kSrcLists)
        if (a.gate && (*a.gate < a.gate_from || *a.gate >= a.gate_to)) return;

    // where the stripe's pixels lie: dense source: byte offset from image n0's first float of the
    // channel; lists: byte offset of the pixel's pointers from image n0's; kOut: outside the image
    int goff[G::IT];
#pragma unroll
    for (int i = 0; i < G::IT; ++i) {
        const int e = i * 64 + lane;
        const int row = div_by(e, a.m_pitch), col = e - row * a.pitch;
        const int ul = u0 - n0 * a.VR + row, dn = div_by(ul, a.m_vr);    // image n0 + dn
        const int iy = ul - dn * a.VR - a.ph, ix = pan * a.SW * a.sw - a.pw + col;
        const bool ok = (e < npx) & (n0 + dn < a.N) & (iy >= 0) & (iy < a.H) & (ix >= 0) & (ix < a.W);
        const int pix = dn * HW + iy * a.W + ix;
        goff[i] = !ok ? kOut : G::SRC == kSrcDense ? (pix + dn * (a.C - 1) * HW) * 4 : pix * a.NCP * 4;
    }
    // a pixel of the tile: row of the panel (from v0 on), column, image and row of the image
    struct Pos { int dv, ox, dn, oy; };
    const int x0 = p0 - v0 * a.SW, y0 = v0 - n0 * a.Ho;
    auto pos_of = [&](int dp) {
        Pos r;
        r.dv = div_by(x0 + dp, a.m_sw);
        r.ox = x0 + dp - r.dv * a.SW;
        r.dn = div_by(y0 + r.dv, a.m_ho);
        r.oy = y0 + r.dv - r.dn * a.Ho;
        return r;
    };
    // LDS byte offset of this lane's B operands, per 16-pixel column block
    int boff[G::NT];
#pragma unroll
    for (int t = 0; t < G::NT; ++t) {
        const int dp = t * 16 + j;
        const Pos r = pos_of(p0 + dp < plast ? dp : plast - p0);
        boff[t] = (((n0 + r.dn) * a.VR + r.oy * a.sh - u0) * a.pitch + r.ox * a.sw + (ks * 4 + q) * a.PL) * 16;
    }

    const int NCH = (a.C + G::CC - 1) / G::CC;
    const int RSn = G::RS ? G::RS : a.R * a.S;
    uint32_t top = 0;

    // ---- staging: load() issues a chunk's global loads, store() puts them into an LDS buffer
    f4v xr[G::SRC == kSrcDense ? G::PPW : 1][G::IT];                        // dense: one pixel's four channels
    constexpr int LI = (G::IT + G::WPS - 1) / G::WPS;                       // lists: items of a wave
    int lb[LI], ln[LI], nb[LI], ne[LI];                                     // where the item's list starts, its length; where the next chunk's starts and ends
    constexpr int LH = (LI + 1) / 2;                                        // (staged in two halves: registers)
    u4v lc[LH][2], lv[LH][2];                                               // its pairs: channels, values
    const int step_w = wave / G::WPS, half_w = wave % G::WPS;
    // (the arrays are addressed from image n0 on with 32-bit byte offsets)
    const int *cp0 = G::SRC == kSrcLists ? a.cptr + (long long)n0 * HW * a.NCP : nullptr;
    const int ebase = G::SRC == kSrcLists ? cp0[0] : 0;
    const __amdgpu_buffer_rsrc_t crs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(a.cidx) + ebase, 0, kOut, 0x00020000);
    const __amdgpu_buffer_rsrc_t vrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.xval) + ebase, 0, kOut, 0x00020000);
    auto load_ptrs = [&](int ci) {
        const int st = ci * (G::CC / kSiCC) + step_w;
        const __amdgpu_buffer_rsrc_t prs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<int *>(cp0) + (st < a.NCP ? st : 0), 0, st < a.NCP ? kOut : 0, 0x00020000);
#pragma unroll
        for (int i = 0; i < LI; ++i) {
            const int off = half_w ? goff[(i * G::WPS + 1) % G::IT] : goff[(i * G::WPS) % G::IT];
            nb[i] = (int)__builtin_amdgcn_raw_buffer_load_b32(prs, off, 0, 0);
            ne[i] = (int)__builtin_amdgcn_raw_buffer_load_b32(prs, off, 4, 0);
        }
    };
    auto take_ptrs = [&]() {
#pragma unroll
        for (int i = 0; i < LI; ++i) {
            lb[i] = nb[i];
            ln[i] = ne[i] - nb[i];
        }
    };
    auto load_dense = [&](int ci) {
#pragma unroll
        for (int pp = 0; pp < G::PPW; ++pp) {
            const int c0 = ci * G::CC + (wave * G::PPW + pp) * 4;
            // from channel c0 of image n0 on; channels past the last one read as zero
            const long long first = ((long long)n0 * a.C + c0) * HW;
            const float *src = a.x + (c0 < a.C ? first : 0);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                // (the condition sits in the descriptor's size: in the offset it becomes a branch)
                const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                    const_cast<float *>(src), 0, c0 + t < a.C ? kOut : 0, 0x00020000);
#pragma unroll
                for (int i = 0; i < G::IT; ++i)
                    xr[pp][i][t] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, goff[i], t * HW * 4, 0));
            }
        }
    };
    auto store_dense = [&](int buf) {
#pragma unroll
        for (int pp = 0; pp < G::PPW; ++pp)
#pragma unroll
            for (int i = 0; i < G::IT; ++i) {
#pragma unroll
                for (int t = 0; t < 4; ++t) see(top, xr[pp][i][t]);
                if (i * 64 + lane < npx)
                    *reinterpret_cast<f4v *>(ldsb + buf * a.buf_bytes + ((wave * G::PPW + pp) * a.PL + i * 64 + lane) * 16) = xr[pp][i];
            }
    };
    // lists: where the item's eight channels lie in the pair arrays (two chunks ahead), the pairs
    // themselves (one chunk ahead); then the eight channels are cleared and the pairs dropped into place
    auto load_lists = [&](int half) {
#pragma unroll
        for (int l = 0; l < LH; ++l)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int i = half * LH + l;
                if (i >= LI) break;
                const int off = ln[i] > h * 4 ? (lb[i] - ebase) * 4 + h * 16 : kOut;
                lc[l][h] = __builtin_amdgcn_raw_buffer_load_b128(crs, off, 0, 0);
                lv[l][h] = __builtin_amdgcn_raw_buffer_load_b128(vrs, off, 0, 0);
            }
    };
    auto store_lists = [&](int half, int buf) {
#pragma unroll
        for (int l = 0; l < LH; ++l) {
            const int i = half * LH + l;
            if (i >= LI) break;
            const int e = (i * G::WPS + half_w) * 64 + lane;
            if (e < npx) {
                char *dst = ldsb + buf * a.buf_bytes + (step_w * 2 * a.PL + e) * 16;
                const f4v z = {0.0f, 0.0f, 0.0f, 0.0f};
                *reinterpret_cast<f4v *>(dst) = z;
                *reinterpret_cast<f4v *>(dst + a.PL * 16) = z;
#pragma unroll
                for (int m = 0; m < kSiCC; ++m)
                    if (m < ln[i]) {
                        const uint32_t c = lc[l][m / 4][m % 4] & 7u;   // (a chunk starts at a multiple of 8)
                        *reinterpret_cast<float *>(dst + (c >> 2) * (uint32_t)(a.PL * 16) + (c & 3u) * 4u) =
                            __uint_as_float(lv[l][m / 4][m % 4]);
                    }
            }
        }
    };

    // ---- A operands of this lane: row k, channels 4q .. 4q+3 of the slice's 16.  3x3: a chunk's nine
    // taps live in registers; as soon as a tap has been multiplied its registers are loaded for the
    // next chunk.  Any other extent: one tap ahead.
    const int krow = kt * 16 * G::MW + mw * 16 + j;
    constexpr int AR = G::RS ? G::RS : 2;
    float av[AR][4];
    const int kb = kt * G::MW + mw;
    // the bank from chunk ci on (packed: of these 16 rows); past the last chunk: nothing
    auto weights = [&](int ci) {
        const long long skip = G::WSRC == kWKC ? (long long)ci * G::CC * 9 : (long long)ci * G::KS * RSn * 256;
        const long long base = G::WSRC == kWKC ? 0 : (long long)kb * a.nslice * RSn * 256;
        const long long size = G::WSRC == kWKC ? (long long)a.K * a.C * 9 : (long long)a.nslice * RSn * 256;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.w) + base + (ci < NCH ? skip : 0), 0,
                                                 ci < NCH ? (int)((size - skip) * 4) : 0, 0x00020000);
    };
    const int wlane = G::WSRC == kWKC ? (krow < a.K ? (krow * a.C + ks * 16 + q * 4) * 36 : kOut)
                                      : ks * RSn * 1024 + lane * 16;
    // K x C x 3 x 3: the lane's 36 consecutive floats of the chunk; floats of channels past the last
    // one belong to the next filter (finite or not, they meet staged zeros, so they are cleared)
    auto load_a_rows = [&](int ci) {
        const int left = a.C - (ci * G::CC + ks * 16 + q * 4);
        float buf[36];
        const __amdgpu_buffer_rsrc_t wrs = weights(ci);
#pragma unroll
        for (int m = 0; m < 9; ++m) {
            const u4v v = __builtin_amdgcn_raw_buffer_load_b128(wrs, wlane + m * 16, 0, 0);
#pragma unroll
            for (int t = 0; t < 4; ++t) buf[m * 4 + t] = __uint_as_float(v[t]);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int rs = 0; rs < 9; ++rs) {
                const float v = t < left ? buf[t * 9 + rs] : 0.0f;
                see(top, v);
                av[rs % AR][t] = v;
            }
    };
    // packed: channels past the last slice lie outside the descriptor and read as zero
    auto load_a_tap = [&](__amdgpu_buffer_rsrc_t wrs, int tap, float (&d)[4]) {
        const u4v v = __builtin_amdgcn_raw_buffer_load_b128(wrs, wlane, tap * 1024, 0);
#pragma unroll
        for (int t = 0; t < 4; ++t) d[t] = __uint_as_float(v[t]);
    };

    f4v acc[G::NT];
#pragma unroll
    for (int t = 0; t < G::NT; ++t) acc[t] = f4v{0.0f, 0.0f, 0.0f, 0.0f};

    // Column blocks are taken in groups of GR whose MFMAs are independent of each other; the B operands
    // of the next group are read while the current one is multiplied.
    constexpr int GR = G::NT < 7 ? G::NT : G::NT == 7 ? 7 : 5, NGR = (G::NT + GR - 1) / GR;
    auto read_group = [&](int B, int tapoff, int t0, f4v (&b)[GR]) {
        int so = B + tapoff;
        asm volatile("" : "+s"(so));   // the sums below are made here, not kept in registers from tap to tap
#pragma unroll
        for (int t = 0; t < GR; ++t)
            if (t0 + t < G::NT) b[t] = *reinterpret_cast<const f4v *>(ldsb + boff[t0 + t] + so);
    };
    auto mul_group = [&](const f4v (&b)[GR], int t0, const float (&w4)[4]) {
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int t = 0; t < GR; ++t)
                if (t0 + t < G::NT)
                    acc[t0 + t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w4[m], b[t][m], acc[t0 + t], 0, 0, 0);
    };

    if constexpr (G::WSRC == kWPacked) {
        if constexpr (G::RS != 0) {
#pragma unroll
            for (int rs = 0; rs < AR; ++rs) load_a_tap(weights(0), rs, av[rs]);
        } else {
            load_a_tap(weights(0), 0, av[0]);
        }
    } else {
        load_a_rows(0);
    }
    if constexpr (G::SRC == kSrcDense) {
        load_dense(0);
        store_dense(0);
    } else {
        load_ptrs(0);
        take_ptrs();
        load_ptrs(1);
        load_lists(0);
        store_lists(0, 0);
        load_lists(1);
        store_lists(1, 0);
    }
    __syncthreads();

    for (int ci = 0; ci < NCH; ++ci) {
        const int B = (ci & 1) * a.buf_bytes;
        // the next chunk's loads are issued without a branch (past the last chunk they fall outside
        // their descriptors and read zeros): behind a branch the compiler cannot count what is in
        // flight, and its waits for A operands would wait for the stripe as well
        if constexpr (G::SRC == kSrcDense) load_dense(ci + 1);
        else {
            take_ptrs();
            load_ptrs(ci + 2);
            load_lists(0);
        }
        // (at two taps of the chunk)
        auto stage_next = [&](int part) {
            if constexpr (G::SRC == kSrcDense) {
                if (part == 0) store_dense((ci + 1) & 1);
            } else {
                store_lists(part, (ci + 1) & 1);
                if (part == 0) load_lists(1);
            }
        };
        if constexpr (G::RS != 0) {
            const __amdgpu_buffer_rsrc_t wnext = weights(ci + 1);
            // (16 waves a CU hide the LDS latency among themselves and have half the registers)
            constexpr int PIPE = G::WAVES < 16 ? 1 : 0;
            f4v b[1 + PIPE][GR];
            read_group(B, 0, 0, b[0]);
            static_for<0, AR * NGR>([&](auto step) {   // (unrolled whatever its size)
                constexpr int st = decltype(step)::value;
                constexpr int rs = st / NGR, gr = st % NGR, up = st + PIPE, nx = up / NGR;
                if (up > 0 && up < AR * NGR) {
                    read_group(B, ((nx / 3) * a.pitch + nx % 3) * 16, (up % NGR) * GR, b[up % (1 + PIPE)]);
                    if (PIPE) __builtin_amdgcn_sched_barrier(0);
                }
                mul_group(b[st % (1 + PIPE)], gr * GR, av[rs]);
                if (gr == NGR - 1) {
                    if (G::WSRC == kWPacked) load_a_tap(wnext, rs, av[rs]);
                    // as late as can be: under load a round trip to memory takes a few microseconds
                    if (rs == (G::SRC == kSrcDense ? 7 : 3)) stage_next(0);
                    if (rs == 7) stage_next(1);
                }
            });
            if (G::WSRC == kWKC) load_a_rows(ci + 1);
        } else {
            int r = 0, s = 0;
            for (int tap = 0; tap < RSn; ++tap) {
                const bool last = tap + 1 == RSn;
                load_a_tap(weights(last ? ci + 1 : ci), last ? 0 : tap + 1, av[1]);
#pragma unroll
                for (int t0 = 0; t0 < G::NT; t0 += GR) {
                    f4v b[GR];
                    read_group(B, (r * a.pitch + s) * 16, t0, b);
                    mul_group(b, t0, av[0]);
                }
#pragma unroll
                for (int t = 0; t < 4; ++t) av[0][t] = av[1][t];
                if (tap == RSn / 2) { stage_next(0); stage_next(1); }
                if (++s == a.S) { s = 0; ++r; }
            }
        }
        __syncthreads();
    }

    // ---- the slices' sums, added in order (the stripe buffers are free)
    if constexpr (G::KS > 1) {
        f4v *red = reinterpret_cast<f4v *>(ldsb);
        if (ks > 0) {
#pragma unroll
            for (int t = 0; t < G::NT; ++t) red[(((ks - 1) * G::MW + mw) * G::NT + t) * 64 + lane] = acc[t];
        }
        __syncthreads();
        if (ks == 0) {
#pragma unroll
            for (int s = 1; s < G::KS; ++s)
#pragma unroll
                for (int t = 0; t < G::NT; ++t) acc[t] += red[(((s - 1) * G::MW + mw) * G::NT + t) * 64 + lane];
        }
    }
    bool bad = top >= 0x7f800000u;
    if (G::WSRC == kWPacked && a.wflag) bad |= *a.wflag != 0;
    const bool slow = __syncthreads_or(bad ? 1 : 0) != 0;
    if (ks != 0) return;

    // ---- bias, activation, store: lane (q, j) holds channels 4q .. 4q+3 of its wave's 16 at pixel j
    const long long plane = (long long)a.Ho * a.Wo;
#pragma unroll
    for (int t = 0; t < G::NT; ++t) {
        const int dp = t * 16 + j;
        const Pos r = pos_of(dp);
        const int n = n0 + r.dn, oy = r.oy, ox = pan * a.SW + r.ox;
        if (p0 + dp > plast || ox >= a.Wo) continue;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const int k = kt * 16 * G::MW + mw * 16 + q * 4 + m;
            if (k >= a.K) continue;
            float v = slow ? slow_output<G>(a, n, k, oy, ox) : acc[t][m];
            if (a.bias) v += a.bias[k];
            a.y[((long long)n * a.K + k) * plane + (long long)oy * a.Wo + ox] = act_apply(v, a.act);
        }
    }
}

// packed copy of a compressed bank (zero-filled before); *flag (likewise): set if an Inf or NaN is met
__global__ void __launch_bounds__(256) pack_rows_kernel(const int *__restrict__ rowptr, const uint32_t *__restrict__ idx,
                                                        const float *__restrict__ val, int RS, int nslice,
                                                        float *__restrict__ packed, int *__restrict__ flag)
{
    const int k = blockIdx.x;
    uint32_t top = 0;
    for (int i = rowptr[k] + (int)threadIdx.x; i < rowptr[k + 1]; i += 256) {
        const int c = (int)(idx[i] / (uint32_t)RS), rs = (int)(idx[i] % (uint32_t)RS);
        see(top, val[i]);
        packed[contract_packed_index(k, c, rs, RS, nslice)] = val[i];
    }
    if (top >= 0x7f800000u) *flag = 1;
}

// packed copy of a dense K x C x 3 x 3 bank, and the copy wT[c][tap][Kpad] the gather kernel reads: a
// work-group takes 16 rows and 16 channels through LDS, so that reads and writes are whole lines.
// *flag: set if an Inf or NaN is met.
__global__ void __launch_bounds__(256) pack_dense_kernel(const float *__restrict__ w, int K, int C, int Kpad, int nslice,
                                                         float *__restrict__ packed, float *__restrict__ wT,
                                                         int *__restrict__ flag)
{
    __shared__ float tile[16][145];
    const int sl = blockIdx.x % nslice, kb = blockIdx.x / nslice, tid = threadIdx.x;
    uint32_t top = 0;
    for (int e = tid; e < 16 * 144; e += 256) {
        const int r = e / 144, f = e % 144, k = kb * 16 + r, c = sl * 16 + f / 9;
        const float v = k < K && c < C ? w[((long long)k * C + sl * 16) * 9 + f] : 0.0f;
        see(top, v);
        tile[r][f] = v;
    }
    if (top >= 0x7f800000u) *flag = 1;
    __syncthreads();
    float *dst = packed + ((long long)kb * nslice + sl) * 9 * 256;
    for (int e = tid; e < 9 * 256; e += 256) {
        const int tap = e / 256, l = (e / 4) % 64, t = e % 4;
        dst[e] = tile[l & 15][((l >> 4) * 4 + t) * 9 + tap];
    }
    for (int e = tid; e < 144 * 16; e += 256) {
        const int f = e / 16, r = e % 16;
        if (sl * 16 + f / 9 < C && kb * 16 + r < Kpad) wT[((long long)sl * 144 + f) * Kpad + kb * 16 + r] = tile[r][f];
    }
}
__global__ void __launch_bounds__(256) clear_kernel(float4 *__restrict__ p, long long n)
{
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
}

// ---------------------------------------------------------------- launch
struct Geo { int MW, KS, NT; };
constexpr Geo kGeo[] = {{4, 2, 13}, {4, 2, 7}, {4, 2, 4}, {4, 4, 4}, {4, 4, 2}, {4, 4, 1}, {2, 4, 4}, {2, 4, 2}};
constexpr int kNGeo = sizeof(kGeo) / sizeof(kGeo[0]);

template <class G> hipError_t launch_cfg(DcArgs a, const ContractPick &p, hipStream_t st)
{
    static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(&contract_kernel<G>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, kLdsMax);
    if (attr != hipSuccess) return attr;
    a.SW = p.SW; a.pitch = p.pitch; a.PL = p.PL; a.buf_bytes = p.buf;
    a.VR = (a.Ho - 1) * a.sh + a.R;
    a.m_pitch = recip_of(a.pitch); a.m_vr = recip_of(a.VR); a.m_sw = recip_of(a.SW); a.m_ho = recip_of(a.Ho);
    a.NKT = (a.K + 16 * G::MW - 1) / (16 * G::MW);
    const long long P = (long long)a.N * a.Ho * a.SW;
    a.tpp = (int)((P + G::T - 1) / G::T);
    const long long nblk = (long long)a.tpp * p.npan * a.NKT;
    if (nblk <= 0 || nblk > 0x7fffffffLL || nblk * G::NTH > 0xffffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(contract_kernel<G>, dim3((unsigned)nblk), dim3(G::NTH), p.lds, st, a);
    return hipGetLastError();
}

template <int SRC, int WSRC, int RS> hipError_t launch_any(const DcArgs &a, const ContractPick &p, hipStream_t st)
{
    switch (p.cfg) {
    case 0: return launch_cfg<DcCfg<4, 2, 13, SRC, WSRC, RS>>(a, p, st);
    case 1: return launch_cfg<DcCfg<4, 2, 7, SRC, WSRC, RS>>(a, p, st);
    case 2: return launch_cfg<DcCfg<4, 2, 4, SRC, WSRC, RS>>(a, p, st);
    case 3: return launch_cfg<DcCfg<4, 4, 4, SRC, WSRC, RS>>(a, p, st);
    case 4: return launch_cfg<DcCfg<4, 4, 2, SRC, WSRC, RS>>(a, p, st);
    case 5: return launch_cfg<DcCfg<4, 4, 1, SRC, WSRC, RS>>(a, p, st);
    case 6: return launch_cfg<DcCfg<2, 4, 4, SRC, WSRC, RS>>(a, p, st);
    case 7: return launch_cfg<DcCfg<2, 4, 2, SRC, WSRC, RS>>(a, p, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace

// The configuration of a launch, by a model of its time in clocks: rounds of work-groups over the 256 CUs, each
// taking per chunk its MFMAs (32 clocks each on four SIMDs; an eighth on top for what the two waves of a SIMD do
// not hide of each other), the staging and a fixed part, then a prologue of one memory round trip and the
// epilogue's stores per 16-pixel column block; then the launch.  Fitted per form to what random geometries took
// (the share that is stored does not matter): 3x3 dense source, strides 1 and 2, 480 launches, standard deviation 5 %;
// other extents (1x1, 5x5, 7x7), 215, 6 %; lists with a packed bank, 350, 4 %; lists with a bank as the caller
// holds it, 350, 5 %.
struct ContractCost {
    double mfma, stage, chunk, round, block, launch;
};
constexpr ContractCost kContractCost[] = {{0.971, 163, 987, 8615, 2747, 3606},     // kContractDense, 3x3
                                          {1.132, 67, 2383, 7345, 2469, 3160},     // kContractDense, any other extent
                                          {1.004, 169, 1378, 4311, 2864, 7213},    // kContractLists
                                          {0.996, 248, 4071, 9309, 2361, 5412}};   // kContractListsRows
ContractPick contract_pick(ContractForm form, int N, int C, int K, int H, int W, int R, int S, int Ho, int Wo, int sh, int sw)
{
    const ContractCost &m = kContractCost[form != kContractDense ? form + 1 : R == 3 && S == 3 ? 0 : 1];
    ContractPick best;
    // weights and the images a stripe can touch are addressed with 32-bit byte offsets, pixels of a
    // panel numbered with ints
    const long long big = 0x7fffffffLL;
    if (4 * contract_packed_elems(K, C, R * S) >= big || (long long)N * Ho * (Wo + 64) >= big || (long long)N * H * W >= big ||
        (long long)N * ((long long)(Ho - 1) * sh + R) >= big || (Ho - 1) * (long long)sh + R > 40000 || Wo > 40000)
        return best;
    double best_clocks = 0;
    int last_npan = 0;
    for (int target : {40000, 64, 48, 32, 24, 16, 12, 8, 6}) {          // widths of a panel
        const int npan0 = (Wo + target - 1) / target, SW = (Wo + npan0 - 1) / npan0, npan = (Wo + SW - 1) / SW;
        if (npan == last_npan) continue;
        last_npan = npan;
        const int pitch = (SW - 1) * sw + S;
        const long long P = (long long)N * Ho * SW;
        for (int g = 0; g < kNGeo; ++g) {
            const Geo &q = kGeo[g];
            const int T = 16 * q.NT;
            const int rows = (T + SW - 2) / SW + 1;             // output rows a tile can touch
            const int cross = (rows - 1 + Ho - 1) / Ho;         // image boundaries among them
            const long long nrow = (long long)(rows - 1) * sh + R + (long long)cross * (R > sh ? R - sh : 0);
            const long long npx = nrow * pitch;
            if (npx > 64 * it_max(q.KS)) continue;
            if ((cross + 2LL) * (C + 8) * H * W * 4 >= big - 64) continue;
            const int PL = (int)((npx + 15) / 16 * 16);
            const int buf = PL * 16 * 4 * q.KS;
            const int red = (q.KS - 1) * q.MW * 64 * q.NT * 16;
            const int lds = 2 * buf > red ? 2 * buf : red;
            if (lds > kLdsMax) continue;
            const long long nwg = (P + T - 1) / T * npan * ((K + 16 * q.MW - 1) / (16 * q.MW));
            const int nch = (C + 16 * q.KS - 1) / (16 * q.KS);
            const double mfma = 36.0 * q.MW * q.NT * q.KS * R * S;
            const double chunk = m.mfma * mfma + m.stage * q.KS * (double)((npx + 63) / 64) + m.chunk;
            const double clocks = (double)((nwg + 255) / 256) * (nch * chunk + m.round + m.block * q.NT) + m.launch;
            if (best.cfg < 0 || clocks < best_clocks) {
                best_clocks = clocks;
                best.cfg = g; best.npan = npan; best.lds = lds;
                best.SW = SW; best.pitch = pitch; best.PL = PL; best.buf = buf;
            }
        }
    }
    best.seconds = best_clocks / 2.4e9;
    return best;
}

hipError_t launch_pack_rows(const int *rowptr, const uint32_t *idx, const float *val, int K, int C, int RS,
                            float *packed, hipStream_t st)
{
    const long long n4 = contract_packed_elems(K, C, RS) / 4 + 1;   // with the flag behind it
    hipLaunchKernelGGL(clear_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, st, reinterpret_cast<float4 *>(packed), n4);
    hipLaunchKernelGGL(pack_rows_kernel, dim3(K), dim3(256), 0, st, rowptr, idx, val, RS, (C + 15) / 16, packed,
                       reinterpret_cast<int *>(packed + (n4 - 1) * 4));
    return hipGetLastError();
}

hipError_t launch_pack_dense(const float *w, int K, int C, int Kpad, float *packed, float *wT, int *flag, hipStream_t st)
{
    const int nslice = (C + 15) / 16;
    hipLaunchKernelGGL(clear_kernel, dim3(1), dim3(256), 0, st, reinterpret_cast<float4 *>(flag), 1LL);
    hipLaunchKernelGGL(pack_dense_kernel, dim3((unsigned)((long long)nslice * (Kpad / 16))), dim3(256), 0, st, w, K, C, Kpad,
                       nslice, packed, wT, flag);
    return hipGetLastError();
}

hipError_t launch_contract_dense(const float *x, const float *packed, const int *wflag, const int *rowptr, const uint32_t *idx,
                                 const float *val, int N, int C, int H, int W, int K, int R, int S, int Ho, int Wo,
                                 int sh, int sw, int ph, int pw, const float *bias, int act, float *y,
                                 const ContractPick &p, hipStream_t st)
{
    if (p.cfg < 0) return hipErrorInvalidValue;
    DcArgs a = {};
    a.x = x; a.w = packed; a.wflag = wflag; a.nslice = (C + 15) / 16; a.rowptr = rowptr; a.idx = idx; a.val = val; a.bias = bias; a.y = y;
    a.N = N; a.C = C; a.H = H; a.W = W; a.K = K; a.R = R; a.S = S; a.Ho = Ho; a.Wo = Wo;
    a.sh = sh; a.sw = sw; a.ph = ph; a.pw = pw; a.act = act;
    if (R == 3 && S == 3) return launch_any<kSrcDense, kWPacked, 9>(a, p, st);
    return launch_any<kSrcDense, kWPacked, 0>(a, p, st);
}

hipError_t launch_contract_lists(const fscnn_input *in, const float *w, const int *wflag, int K, int Ho,
                                 int Wo, int ph, int pw, const float *bias, int relu, float *y,
                                 const ContractPick &p, const int *gate, int gate_from, int gate_to, hipStream_t st)
{
    if (p.cfg < 0 || in->CC != kSiCC) return hipErrorInvalidValue;
    DcArgs a = {};
    a.gate = gate; a.gate_from = gate_from; a.gate_to = gate_to; a.cptr = in->cptr; a.cidx = in->cidx; a.xval = in->xval; a.NCP = in->NCH;
    a.w = w; a.nslice = (in->C + 15) / 16; a.wflag = wflag; a.bias = bias; a.y = y;
    a.N = in->N; a.C = in->C; a.H = in->H; a.W = in->W; a.K = K; a.R = 3; a.S = 3; a.Ho = Ho; a.Wo = Wo;
    a.sh = a.sw = 1; a.ph = ph; a.pw = pw; a.act = relu;
    if (wflag) return launch_any<kSrcLists, kWPacked, 9>(a, p, st);
    return launch_any<kSrcLists, kWKC, 9>(a, p, st);
}

}  // namespace fscnn
