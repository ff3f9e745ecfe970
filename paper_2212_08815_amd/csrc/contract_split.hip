// Convolution as a dense contraction on the matrix cores, fp32 operands taken apart into three bfloat16 parts.
//
// A float is the exact sum of three bfloat16 numbers (8 + 8 + 8 bits, each part the previous remainder rounded
// to nearest; operands are multiplied by 2^16 first, so that subnormal ones have their parts too), and a product of two
// floats is, up to 2^-24 of it (root mean square 2^-27.4), the six products of parts h*h, h*m, m*h, m*m, h*l, l*h.  v_mfma_f32_32x32x16_bf16
// multiplies at 2.1 PFLOP/s on this chip (registers only), so six of them make 350 TFLOP/s of fp32-like
// products where v_mfma_f32_16x16x4_f32 (contract.hip) makes 154.  Precision: the matrix unit cuts what it adds
// two bits below the accumulator's last one, towards zero, which biases a sum that all six products go into (512
// channels, 3x3: 6.3e-7 of the result in 2-norm, mean -1e-7, against 4.4e-7 of the fp32 unit).  So h*h has an
// accumulator of its own and the five small products share another one, 2^-8 of its size, added at the end: 1.7e-7.
// Sums of one sign are no worse off: 4608 products of magnitudes, 512 -> 512 at 28x28, N = 8: 1.8e-7, mean -7e-10 of the
// result (the fp32 unit: 3.6e-7); a bank that averages: 1.7e-7 (4.4e-7).  Sums of one to three products are the less exact ones here (up to 1.05
// times the 2-norm error of one rounding each, a single product up to 1.5 times the largest): splits() in api.hip keeps such filters out.
//
// How it is mapped (numbering of pixels, panels and stripes as in contract.hip):
//   * output channels are the rows of the product, output pixels its columns.  A work-group owns 32*MW channels and
//     T = 32*NB pixels; of its MW*KS*NW waves (eight), MW lie along the channels (32 rows each), KS take a 16-channel
//     slice each of every chunk of 16*KS input channels, NW divide the pixel blocks.
//   * LDS holds the stripe as [octet of channels][pixel][part][8 channels]: 48 bytes per pixel and octet, so that one
//     ds_read_b128 is the B operand of a part, and consecutive pixels fall on different banks (3 is coprime to 16).
//     Two buffers, one barrier per chunk: a chunk's stores are spread over the steps of the chunk before, four
//     pixels of one octet by lane, whose 16-byte loads were issued a chunk earlier.  Pixels outside the image are
//     cleared once.
//   * Units.  Groups of four images in an N4 tensor are one image with rows of W x 4 columns, pixel (x, image b of the group) in column
//     4x + b: a tap to the right is four columns away, everything else is as it was (N4 into NCHW differs in the stores alone).
//     With the merged pool the pixels are numbered by units of 2x2: a block of 32 is 16 adjacent columns of two rows, 8 units, so
//     that a unit's maximum is taken over four lanes and reads of B stay as free of bank conflicts as they were.  Without it a unit
//     is a pixel.  4x4 images, 512 -> 1024, N = 18, 16 % stored, N4: 448 us gathered (a 16x16 tile holds one image), 27 so; 52 layers
//     on 128x128, N = 18: 3638 -> 1253; 13 layers at 128x128, N = 12, 10 %: 724 -> 558.  250 random layers through N4 tensors or
//     with the pool, 3 to 50 % stored: 1.29 times as fast as gathered, where the faster of the two each time would make 1.30.
//   * where a launch leaves CUs idle the chunks are divided over several work-groups per tile, and a second launch adds up.
//   * the A operands go from global memory to registers a few taps ahead, packed as the lanes want them:
//     [32 rows][16 channels][tap][part][lane][8].
// What bounds it (512 -> 512 at 28x28, N = 8, 131 us; before, in fp32, 252): the matrix instructions, 104 us with the loads, splits and
// stores of the chunks left out, an eighth of the CUs without a tile; staging adds 20, the loads of A operands 7.  Its estimate is at kSplitCost below.
//
// A compressed activation is served from the dense form its handle keeps (si_choose in conv_si.hip says when), with a
// dense 3x3 bank taken apart as it is prepared or, where the caller holds it, before the launch.
//
// Non-finite operands: a value that is Inf, NaN or has an infinite first part (from 2^112 on) has a NaN last part, so every
// output it is multiplied into (zeros included) is NaN; an output that is not finite (a sum from 2^96 on among them) is made
// again entry by entry, from stored entries only (0 * Inf cannot appear): 2.4 ms where all of 128 -> 128 at 28x28, N = 8 are.
#include <type_traits>

#include "internal.h"
#include "lds_dma.h"

namespace fscnn {

namespace {

typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f2v __attribute__((ext_vector_type(2)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef __bf16 bf2v __attribute__((ext_vector_type(2)));

constexpr int kLdsMax = 160 * 1024 - 512;
constexpr int kOut = 0x7ffffff0;         // beyond any descriptor's range: the buffer load returns 0

// where an output that is not finite is made again from
struct SlowArgs {
    const int *rowptr;                   // filter rows and a dense x, or (NULL)
    const uint32_t *idx;
    const float *val;
    const int *cptr;                     // lists and a dense bank
    const uint32_t *cidx;
    const float *xval;
    int NCP;
    const float *w;                      // w[k*wk + c*wc + tap*wt]
    int wk, wc, wt;
};

struct SpArgs {
    const float *x;
    const char *w;
    const float *bias;
    float *y;
    const int *gate;                     // if not NULL and *gate < gate_from, another kernel serves the call
    int gate_from;
    // N, W, pw: groups of images; columns and padding times the images of a group.  Hu, Wu: rows and columns of units (see the top)
    int N, C, H, W, K, nslice, nkb, Hu, Wu, sh, sw, ph, pw, act;
    int SW, tpp, pitch, PL, VR, NKT, QPR, buf_bytes;
    int parts, cpp, nblk;                // the chunks are divided over `parts` work-groups per tile, cpp each; tiles
    float *sums;                         // parts > 1: where they leave their sums, each part in the order of y
    uint32_t m_qpr, m_vr, m_sw, m_ho;    // reciprocals for div_by()
    SlowArgs slow;
    // (behind what all launches read: the arguments come a line at a time, from memory)
    int ystep, rext;                     // input rows from a unit to the one below, and of a unit
    int il, pool, out4, images;          // log2 of the images of a group; merged pool; y is N4; images in all
};

// x / d for a divisor whose reciprocal ceil(2^31 / d) the host computed; exact while x * d < 2^31
__device__ inline int div_by(int x, uint32_t m) { return (int)__umulhi((uint32_t)x * 2u, m); }
inline uint32_t recip_of(int d) { return (uint32_t)(((1LL << 31) + d - 1) / d); }

// The parts of two floats times kScale, packed in pairs.  The smallest bfloat16 is 2^-133, the smallest float 2^-149: so no
// operand loses bits, and a sum is divided by kScale^2 at its end
constexpr float kScale = 65536.0f, kUnscale = 1.0f / 65536.0f / 65536.0f;
__device__ __forceinline__ void split2(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l)
{
    a *= kScale; b *= kScale;
    h = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2v{a, b}, bf2v));
    const float ra = a - __uint_as_float(h << 16), rb = b - __uint_as_float(h & 0xffff0000u);
    m = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2v{ra, rb}, bf2v));
    const float la = ra - __uint_as_float(m << 16), lb = rb - __uint_as_float(m & 0xffff0000u);
    l = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2v{la, lb}, bf2v));
}

template <int MW_, int KS_, int NW_, int NB_, int R_, bool GEN_> struct SpCfg {
    static constexpr int MW = MW_, KS = KS_, NW = NW_, NB = NB_, R = R_, RS = R * R;
    static constexpr bool GEN = GEN_;                            // N4 tensors or the merged pool
    static constexpr int WAVES = MW * KS * NW, NTH = WAVES * 64;
    static constexpr int CC = 16 * KS, OCT = 2 * KS;             // channels and octets per chunk
    static constexpr int T = 32 * NB;
    static constexpr int NT = (NB + NW - 1) / NW;                // pixel blocks of a wave (the last one may have fewer)
    static constexpr int SETS = R == 3 ? 3 : 5;                  // taps whose A operands are loaded or in use
    static constexpr int WPO = WAVES / OCT;                      // waves that stage one octet
    static constexpr int QMAX = 64 * WPO;                        // items (rows x quads of pixels) of a stripe, at most
    static constexpr int RED_BYTES = KS > 1 ? WAVES * NT * 64 * 64 : 0;
    static_assert(WAVES == 8 && WPO * OCT == WAVES && RS % SETS == 0, "layout of the work-group");
};

template <int I, int N, class F> __device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// one output, in row oy and column x of output group n (column and image of the group, for N4 tensors)
template <int R> __device__ float slow_output(const SpArgs &a, int n, int k, int oy, int x)
{
    constexpr int RS = R * R;
    const SlowArgs &s = a.slow;
    const int W = a.W >> a.il, pw = a.pw >> a.il, ox = x >> a.il, img = x - (ox << a.il);
    double acc = 0.0;                                 // (one chain of thousands of sums)
    if (s.rowptr) {
        const float *xn = a.x + (long long)n * a.C * a.H * a.W + img;
        for (int i = s.rowptr[k]; i < s.rowptr[k + 1]; ++i) {
            const uint32_t f = s.idx[i];
            const int c = (int)(f / RS), rs = (int)(f % RS);
            const int iy = oy * a.sh - a.ph + rs / R, ix = ox * a.sw - pw + rs % R;
            if (iy >= 0 && iy < a.H && ix >= 0 && ix < W)
                acc = __builtin_fma((double)s.val[i], (double)xn[((long long)c * a.H + iy) * a.W + (ix << a.il)], acc);
        }
    } else {
        for (int rs = 0; rs < RS; ++rs) {
            const int iy = oy * a.sh - a.ph + rs / R, ix = ox * a.sw - pw + rs % R;
            if (iy < 0 || iy >= a.H || ix < 0 || ix >= W) continue;
            const long long pix = ((long long)n * a.H + iy) * W + ix;   // (lists: NCHW)
            for (int i = s.cptr[pix * s.NCP]; i < s.cptr[(pix + 1) * s.NCP]; ++i)
                acc = __builtin_fma((double)s.xval[i], (double)s.w[(long long)k * s.wk + (long long)s.cidx[i] * s.wc + (long long)rs * s.wt], acc);
        }
    }
    return (float)acc;
}

// 2x2 max-pool over four lanes that hold a unit's results, (0, 0) (0, 1) (1, 0) (1, 1) by dy, dx: rows first, as the gather kernels do
__device__ __forceinline__ float pool4(float v, int dx, int dy, int dxbit)
{
    const float o = __shfl_xor(v, 16, 64);
    const float r0 = dy ? o : v, r1 = dy ? v : o, m = r1 > r0 ? r1 : r0;
    const float p = __shfl_xor(m, dxbit, 64);
    const float c0 = dx ? p : m, c1 = dx ? m : p;
    return c1 > c0 ? c1 : c0;
}

// one wave's part: NT blocks of 32 pixels
template <class G, int NT> __device__ __forceinline__ void split_body(const SpArgs &a, char *ldsb, const int wave, const int lane)
{
    const int mw = wave % G::MW, ks = wave / G::MW % G::KS, nw = wave / (G::MW * G::KS);
    const int j = lane & 31, q = lane >> 5;
    const int part = a.parts > 1 ? blockIdx.x / a.nblk : 0, blk = blockIdx.x - part * a.nblk;
    const int kt = blk % a.NKT, tile = blk / a.NKT;
    const int pan = tile / a.tpp;
    const int il = G::GEN ? a.il : 0;
    const bool pool = G::GEN && a.pool;
    const int TU = pool ? G::T / 4 : G::T;            // units of a tile
    const int p0 = (tile % a.tpp) * TU;
    const int ptot = a.N * a.Hu * a.SW;               // units of a panel
    const int plast = p0 + TU < ptot ? p0 + TU - 1 : ptot - 1;
    const int HW = a.H * a.W;
    const int ystep = G::GEN ? a.ystep : a.sh;
    auto virt = [&](int v) { return (v / a.Hu) * a.VR + (v % a.Hu) * ystep; };   // first input row of row v of units
    const int v0 = p0 / a.SW;
    const int u0 = virt(v0), nrow = virt(plast / a.SW) + (G::GEN ? a.rext : G::R) - u0;
    const int n0 = v0 / a.Hu;
    // this part's chunks; channels from cend on read as zero
    const int CI0 = part * a.cpp, NCH = (a.C + G::CC - 1) / G::CC < CI0 + a.cpp ? (a.C + G::CC - 1) / G::CC : CI0 + a.cpp;
    const int cend = a.C < NCH * G::CC ? a.C : NCH * G::CC;
    if (a.gate && *a.gate < a.gate_from) return;

    // ---- staging: an item is four pixels of a stripe's row (the last ones of a row overlap the ones before), eight channels of each
    const int oct = wave / G::WPO;
    int goff = kOut, lpx = -1;                        // byte offset from image n0's first float of the channel; pixel in the stripe
    {
        const int e = (wave % G::WPO) * 64 + lane;
        const int row = div_by(e, a.m_qpr), quad = e - row * a.QPR;
        const int ul = u0 - n0 * a.VR + row, dn = div_by(ul, a.m_vr);    // image n0 + dn
        const int iy = ul - dn * a.VR - a.ph, c0 = pan * a.SW * (pool ? 2 * a.sw : a.sw) - a.pw;
        const int first = c0 > 0 ? c0 : 0, end = c0 + a.pitch < a.W ? c0 + a.pitch : a.W;   // the row's columns in the image: 4 or more
        const int ix = first + quad * 4 + 4 <= end ? first + quad * 4 : end - 4;
        if (row < nrow && n0 + dn < a.N && iy >= 0 && iy < a.H) {
            goff = (dn * a.C * HW + iy * a.W + ix) * 4;
            lpx = row * a.pitch + ix - c0;
        }
    }
    f4v xr[8];
    auto load_x = [&](int ci) {
        const int c0 = ci * G::CC + oct * 8;
        // from channel c0 of image n0 on; channels past the last one read as zero
        const float *src = a.x + (c0 < cend ? ((long long)n0 * a.C + c0) * HW : 0);
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            // (the condition sits in the descriptor's size: in the offset it becomes a branch)
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(src), 0, c0 + t < cend ? kOut : 0, 0x00020000);
            xr[t] = __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(rs, goff, t * HW * 4, 0));
        }
    };
    auto store_x = [&](int buf, auto pixel) {         // one of the four pixels
        constexpr int px = decltype(pixel)::value;
        u4v h, m, l;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            uint32_t hh, mm, ll;
            split2(xr[2 * t][px], xr[2 * t + 1][px], hh, mm, ll);
            h[t] = hh; m[t] = mm; l[t] = ll;
        }
        if (lpx >= 0) {
            u4v *d = reinterpret_cast<u4v *>(ldsb + buf + (oct * a.PL + lpx + px) * 48);
            d[0] = h; d[1] = m; d[2] = l;
        }
    };

    // a unit of the tile: column, image group (from n0 on) and row of the image
    struct Pos { int ox, dn, oy; };
    const int x0 = p0 - v0 * a.SW, y0 = v0 - n0 * a.Hu;
    auto pos_of = [&](int dp) {
        Pos r;
        const int dv = div_by(x0 + dp, a.m_sw);
        r.ox = x0 + dp - dv * a.SW;
        r.dn = div_by(y0 + dv, a.m_ho);
        r.oy = y0 + dv - r.dn * a.Hu;
        return r;
    };
    // this lane's unit in a block of 32 pixels, and its place in a unit of 2x2: 16 adjacent columns of two rows
    const int dxbit = il ? 4 : 1, dx = pool && (j & dxbit), dy = pool ? j >> 4 : 0;
    const int ju = !pool ? j : il ? (j & 3) | (j >> 1 & 4) : j >> 1 & 7;
    auto unit_of = [&](int t) { return (nw * G::NT + t) * (pool ? 8 : 32) + ju; };
    // LDS byte offset of this lane's B operands, per block
    int boff[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int du = unit_of(t);
        const Pos r = pos_of(p0 + du < plast ? du : plast - p0);
        int row = (n0 + r.dn) * a.VR + r.oy * ystep - u0, col = r.ox * a.sw;
        if constexpr (G::GEN) {
            const int ox = r.ox >> il;
            row += dy * a.sh;
            col = (((pool ? 2 * ox + dx : ox) * a.sw) << il) + r.ox - (ox << il);
        }
        boff[t] = (row * a.pitch + col + (ks * 2 + q) * a.PL) * 48;
    }
    constexpr int NS = G::RS * NT;                    // steps of a chunk: (tap, block)
    // blocks whose B operands are requested or in use (a divisor of the steps, so that every step's registers are fixed)
    constexpr int D = NT >= 4 ? 2 : NS % 3 == 0 ? 3 : NS % 2 == 0 ? 2 : 5;
    static_assert(NS % D == 0, "ring of B operands");
    u4v b[D][3];
    auto read_b = [&](int buf, auto step) {
        constexpr int st = decltype(step)::value, tap = st / NT;
        int so = buf + ((tap / G::R) * a.pitch + ((tap % G::R) << il)) * 48;
        asm volatile("" : "+s"(so));                  // the sum below is made here, not kept in registers from tap to tap
        const u4v *s = reinterpret_cast<const u4v *>(ldsb + boff[st % NT] + so);
#pragma unroll
        for (int p = 0; p < 3; ++p) b[st % D][p] = s[p];
    };

    // ---- A operands: this wave's 32 rows, its slice of chunk ci (rows and slices past the last read as zero)
    const int kb = kt * G::MW + mw;
    auto weights = [&](int ci) {
        const bool ok = kb < a.nkb && (ci * G::KS + ks) * 16 < cend;
        const long long at = ((long long)kb * a.nslice + ci * G::KS + ks) * (G::RS * 3072);
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(a.w) + (ok ? at : 0), 0, ok ? G::RS * 3072 : 0, 0x00020000);
    };
    u4v av[G::SETS][3];
    auto load_a = [&](__amdgpu_buffer_rsrc_t rs, int tap, u4v (&d)[3]) {
#pragma unroll
        for (int p = 0; p < 3; ++p) d[p] = __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, tap * 3072 + p * 1024, 0);
    };

    f16v big[NT], small[NT];                          // sums of h*h, and of the five other products
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) big[t][i] = small[t][i] = 0.0f;
    auto multiply = [&](const u4v (&w)[3], auto step) {
        constexpr int st = decltype(step)::value, t = st % NT;
        constexpr int WP[5] = {1, 0, 2, 0, 1}, XP[5] = {1, 2, 0, 1, 0};   // m*m h*l l*h h*m m*h
#pragma unroll
        for (int m = 0; m < 5; ++m)
            small[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8v, w[WP[m]]), __builtin_bit_cast(bf8v, b[st % D][XP[m]]),
                                                               small[t], 0, 0, 0);
        big[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8v, w[0]), __builtin_bit_cast(bf8v, b[st % D][0]), big[t], 0, 0, 0);
    };

    {
        const __amdgpu_buffer_rsrc_t w0 = weights(CI0);
#pragma unroll
        for (int s = 0; s < G::SETS; ++s) load_a(w0, s, av[s]);
    }
    load_x(CI0);
    for (int e = wave * 64 + lane; e * 16 < 2 * a.buf_bytes; e += G::NTH) reinterpret_cast<u4v *>(ldsb)[e] = u4v{0, 0, 0, 0};
    lds_only_barrier();
    static_for<0, 4>([&](auto px) { store_x(0, px); });
    lds_only_barrier();
    static_for<0, D - 1>([&](auto st) { read_b(0, st); });
    // the next chunk's pixels are stored at steps LAST-3 .. LAST (several a step where a chunk is short); after LAST
    // comes the barrier, and then the first reads of the next chunk
    constexpr int LAST = NS - D, FIRST = LAST >= 3 ? LAST - 3 : 0, PER = (4 + LAST - FIRST) / (LAST + 1 - FIRST);
    int cur = 0;
    for (int ci = CI0; ci < NCH; ++ci) {
        const int nxt = a.buf_bytes - cur;
        // (past the last chunk all loads fall outside their descriptors and read zeros: no branches, behind which
        // the compiler could not count what is in flight)
        const __amdgpu_buffer_rsrc_t wcur = weights(ci), wnext = weights(ci + 1);
        static_for<0, NS>([&](auto step) {
            constexpr int st = decltype(step)::value, tap = st / NT;
            if constexpr (st == LAST + 1) lds_only_barrier();
            read_b(st + D - 1 < NS ? cur : nxt, std::integral_constant<int, (st + D - 1) % NS>{});
            __builtin_amdgcn_sched_barrier(0);
            multiply(av[tap % G::SETS], step);
            if constexpr (st % NT == NT - 1) {
                constexpr int up = tap + G::SETS;
                load_a(up < G::RS ? wcur : wnext, up % G::RS, av[tap % G::SETS]);
            }
            if constexpr (st >= FIRST && st <= LAST) {
                static_for<0, PER>([&](auto i) {
                    constexpr int px = (st - FIRST) * PER + decltype(i)::value;
                    if constexpr (px < 4) store_x(nxt, std::integral_constant<int, px>{});
                });
            }
            if constexpr (st == 0) load_x(ci + 1);
        });
        cur = nxt;
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) big[t] += small[t];

    // ---- the slices' sums, added in order: wave ks finishes registers ks*OWN .. of its blocks
    constexpr int OWN = 16 / G::KS;
    float own[NT][OWN];
    if constexpr (G::KS > 1) {
        __syncthreads();                              // (the stripe buffers are free)
        f4v *red = reinterpret_cast<f4v *>(ldsb);
        auto at = [&](int from, int to, int t, int v) {
            return ((((nw * G::MW + mw) * G::KS + from) * G::KS + to) * G::NT + t) * (OWN / 4 * 64) + v * 64 + lane;
        };
#pragma unroll
        for (int s = 0; s < G::KS; ++s) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int v = 0; v < OWN / 4; ++v) {
                    const int r = s * OWN + v * 4;
                    const f4v z = {big[t][r], big[t][r + 1], big[t][r + 2], big[t][r + 3]};
                    red[at(ks, s, t, v)] = z;
                }
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < OWN / 4; ++v) {
                f4v sum = red[at(0, ks, t, v)];
#pragma unroll
                for (int s = 1; s < G::KS; ++s) sum += red[at(s, ks, t, v)];
#pragma unroll
                for (int i = 0; i < 4; ++i) own[t][v * 4 + i] = sum[i];
            }
    } else {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) own[t][i] = big[t][i];
    }

    // ---- bias, activation, store: register r of lane (q, j) is row 8*(r/4) + 4*q + r%4 at pixel j
    const long long plane = (long long)a.Hu * a.Wu;
    auto row_of = [&](int i) {
        const int r = ks * OWN + i;
        return kb * 32 + 8 * (r >> 2) + 4 * q + (r & 3);
    };
    // whether the lane's unit of block t is one, and where its results go (row 0 of the product; kp from there to the next).  Groups
    // of four images go into an NCHW tensor each to its own
    auto exists = [&](int t, const Pos &r) { return p0 + unit_of(t) <= plast && pan * a.SW + r.ox < a.Wu; };
    const bool apart = G::GEN && il && !a.out4;
    const long long kp = apart ? plane >> 2 : plane;
    auto dest = [&](const Pos &r) {
        const int xu = pan * a.SW + r.ox;
        if (apart) return a.y + ((n0 + r.dn) * 4 + (xu & 3)) * (a.K * kp) + (long long)r.oy * (a.Wu >> 2) + (xu >> 2);
        return a.y + (long long)(n0 + r.dn) * a.K * plane + (long long)r.oy * a.Wu + xu;
    };
    // (what images past the last one of an N4 tensor hold is nobody's concern)
    auto real = [&](const Pos &r) { return !il || (n0 + r.dn) * 4 + ((pan * a.SW + r.ox) & 3) < a.images; };
    if (a.parts > 1) {                                // parts_finish_kernel does the rest
        const int per = pool ? 4 : 1;                 // (a unit's results side by side)
        float *to = a.sums + part * (a.N * a.K * plane * per);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const Pos r = pos_of(unit_of(t));
            if (!exists(t, r)) continue;
            float *y = to + ((long long)(n0 + r.dn) * a.K * plane + (long long)r.oy * a.Wu + pan * a.SW + r.ox) * per + 2 * dy + dx;
#pragma unroll
            for (int i = 0; i < OWN; ++i)
                if (row_of(i) < a.K) y[row_of(i) * plane * per] = own[t][i] * kUnscale;
        }
        return;
    }
    bool finite = true;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const Pos r = pos_of(unit_of(t));
        if (!exists(t, r) || (apart && !real(r))) continue;
        float *y = dest(r);
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
            const int k = row_of(i);
            if (k >= a.K) continue;
            float v = own[t][i] * kUnscale;
            finite &= __builtin_fabsf(v) < __builtin_inff() || !real(r);
            if (pool) v = pool4(v, dx, dy, dxbit);
            if (a.bias) v += a.bias[k];
            if (!pool || !(dx | dy)) y[(long long)k * kp] = act_apply(v, a.act);
        }
    }
    if (pool) {                                       // a unit's four lanes go on together
        finite = __shfl_xor((int)finite, 16, 64) && finite;
        finite = __shfl_xor((int)finite, dxbit, 64) && finite;
    }
    if (finite) return;
#pragma nounroll
    for (int o = 0; o < NT * OWN; ++o) {              // (a lane's own stores: in order)
        const int t = o / OWN, k = row_of(o % OWN);
        const Pos r = pos_of(unit_of(t));
        if (!exists(t, r) || (apart && !real(r)) || k >= a.K) continue;
        const int xu = pan * a.SW + r.ox, ox = xu >> il;
        float v = pool ? slow_output<G::R>(a, n0 + r.dn, k, 2 * r.oy + dy, ((2 * ox + dx) << il) + xu - (ox << il))
                       : slow_output<G::R>(a, n0 + r.dn, k, r.oy, xu);
        if (pool) v = pool4(v, dx, dy, dxbit);
        if (a.bias) v += a.bias[k];
        if (!pool || !(dx | dy)) dest(r)[(long long)k * kp] = act_apply(v, a.act);
    }
}

template <class G> __global__ void __launch_bounds__(G::NTH, 2) split_kernel(const SpArgs a)
{
    extern __shared__ __align__(256) char ldsb[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr int LAST_NT = G::NB - (G::NW - 1) * G::NT;
    if (LAST_NT == G::NT || wave < G::MW * G::KS * (G::NW - 1)) split_body<G, G::NT>(a, ldsb, wave, lane);
    else split_body<G, LAST_NT>(a, ldsb, wave, lane);
}

// Sums of the parts, in their order.  Bound by the launch and by one round trip to the last-level cache (512 x 14 x 14 in 4 parts: 2 us).
template <int R, bool POOL> __global__ void __launch_bounds__(256) parts_finish_kernel(const SpArgs a)
{
    constexpr int PER = POOL ? 4 : 1;                  // results of a unit
    typedef float vec __attribute__((ext_vector_type(PER)));
    const long long plane = (long long)a.Hu * a.Wu, total = a.N * a.K * plane, i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    const vec *s = reinterpret_cast<const vec *>(a.sums) + i;
    float v[PER] = {};
    for (int p0 = 0; p0 < a.parts; p0 += 8) {          // eight loads in flight
        vec u[8];
#pragma unroll
        for (int p = 0; p < 8; ++p) u[p] = p0 + p < a.parts ? s[(p0 + p) * total] : vec(0.0f);
#pragma unroll
        for (int p = 0; p < 8; ++p)
#pragma unroll
            for (int e = 0; e < PER; ++e) v[e] += u[p][e];
    }
    const long long nk = i / plane;
    const int k = (int)(nk % a.K), n = (int)(nk / a.K), o = (int)(i - nk * plane), oy = o / a.Wu, xu = o % a.Wu, ox = xu >> a.il;
    const int img = a.il ? n * 4 + (xu & 3) : 0;
    float m = 0.0f;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        if (!(__builtin_fabsf(v[e]) < __builtin_inff()) && img < a.images)
            v[e] = POOL ? slow_output<R>(a, n, k, 2 * oy + e / 2, ((2 * ox + e % 2) << a.il) + xu - (ox << a.il)) : slow_output<R>(a, n, k, oy, xu);
    }
    if constexpr (POOL) {
        const float c0 = v[2] > v[0] ? v[2] : v[0], c1 = v[3] > v[1] ? v[3] : v[1];
        m = c1 > c0 ? c1 : c0;
    } else {
        m = v[0];
    }
    if (a.bias) m += a.bias[k];
    m = act_apply(m, a.act);
    if (!a.il || a.out4) a.y[i] = m;
    else if (img < a.images) a.y[((long long)img * a.K + k) * (plane >> 2) + (long long)oy * (a.Wu >> 2) + ox] = m;
}

// ---------------------------------------------------------------- packed banks

// of compressed filters: a work-group puts the entries of 32 rows and 16 channels together in LDS, zeros between them, so that the bank
// is written once, in whole lines (cleared and scattered before: 512 x 512, 10 % stored, 14.2 MB: 12 to 13 us as two launches, 8.9 so)
template <int RS> __global__ void __launch_bounds__(512) split_rows_kernel(const int *__restrict__ rowptr, const uint32_t *__restrict__ idx,
                                                                          const float *__restrict__ val, int K, int nslice, u4v *__restrict__ out)
{
    constexpr int ROW = 16 * RS + 1;                  // (odd: rows fall on different banks)
    __shared__ float tile[32 * ROW];
    const int sl = blockIdx.x % nslice, kb = blockIdx.x / nslice;
    for (int e = threadIdx.x; e < 32 * ROW; e += 512) tile[e] = 0.0f;
    __syncthreads();
    // 16 lanes a row: the first entry of the slice by bisection (entries ascend), then the entries
    const int r = threadIdx.x / 16, k = kb * 32 + r;
    if (k < K) {
        const uint32_t from = (uint32_t)sl * 16 * RS, to = from + 16 * RS;
        int lo = rowptr[k], hi = rowptr[k + 1];
        const int end = hi;
        while (lo < hi) {
            const int mid = lo + (hi - lo) / 2;
            if (idx[mid] < from) lo = mid + 1; else hi = mid;
        }
        for (int i = lo + (int)(threadIdx.x % 16); i < end; i += 16) {
            const uint32_t f = idx[i];
            if (f >= to) break;
            tile[r * ROW + (int)(f - from)] = val[i];
        }
    }
    __syncthreads();
    u4v *dst = out + (long long)blockIdx.x * (RS * 192);
    for (int e = threadIdx.x; e < RS * 64; e += 512) {
        const int tap = e / 64, lane = e % 64;
        const float *src = &tile[(lane & 31) * ROW + (lane >> 5) * 8 * RS + tap];
        u4v h, m, l;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            uint32_t hh, mm, ll;
            split2(src[2 * t * RS], src[(2 * t + 1) * RS], hh, mm, ll);
            h[t] = hh; m[t] = mm; l[t] = ll;
        }
        dst[tap * 192 + lane] = h; dst[tap * 192 + 64 + lane] = m; dst[tap * 192 + 128 + lane] = l;
    }
}
// of a dense K x C x 3 x 3 bank: a work-group takes 32 rows and 16 channels through LDS, so that reads and writes are whole lines
// (512 x 512: 9.4 MB read, 14.2 written).  One (tap, lane) per thread: 256 x 256 in 8.7 us with 256 threads, 5.2 so
constexpr int kBankThreads = 9 * 64;
__global__ void __launch_bounds__(kBankThreads) split_dense_kernel(const float *__restrict__ w, int K, int C, int nslice, u4v *__restrict__ out)
{
    __shared__ float tile[32][145];
    const int sl = blockIdx.x % nslice, kb = blockIdx.x / nslice;
    for (int e = threadIdx.x; e < 32 * 144; e += kBankThreads) {
        const int r = e / 144, f = e % 144, k = kb * 32 + r, c = sl * 16 + f / 9;
        tile[r][f] = k < K && c < C ? w[((long long)k * C + sl * 16) * 9 + f] : 0.0f;
    }
    __syncthreads();
    u4v *dst = out + (long long)blockIdx.x * (9 * 192);
    const int tap = threadIdx.x / 64, lane = threadIdx.x % 64;
    const float *src = &tile[lane & 31][(lane >> 5) * 72 + tap];
    u4v h, m, l;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        uint32_t hh, mm, ll;
        split2(src[t * 18], src[t * 18 + 9], hh, mm, ll);
        h[t] = hh; m[t] = mm; l[t] = ll;
    }
    dst[tap * 192 + lane] = h; dst[tap * 192 + 64 + lane] = m; dst[tap * 192 + 128 + lane] = l;
}

// ---------------------------------------------------------------- launch
struct Geo { int MW, KS, NW, NB; };
constexpr Geo kGeo[] = {{2, 2, 2, 7}, {2, 2, 2, 6}, {2, 2, 2, 5}, {2, 2, 2, 4}, {2, 2, 2, 3}, {4, 2, 1, 4}, {4, 2, 1, 3}, {4, 2, 1, 2},
                        {2, 4, 1, 2}, {2, 4, 1, 1}};
constexpr int kNGeo = sizeof(kGeo) / sizeof(kGeo[0]);

template <class G> hipError_t launch_cfg(SpArgs a, const ContractPick &p, hipStream_t st)
{
    static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(&split_kernel<G>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, kLdsMax);
    if (attr != hipSuccess) return attr;
    a.SW = p.SW; a.pitch = p.pitch; a.PL = p.PL; a.buf_bytes = p.buf; a.QPR = p.qpr;
    a.VR = (a.Hu - 1) * a.ystep + a.rext;
    a.m_qpr = recip_of(a.QPR); a.m_vr = recip_of(a.VR); a.m_sw = recip_of(a.SW); a.m_ho = recip_of(a.Hu);
    a.NKT = (a.K + 32 * G::MW - 1) / (32 * G::MW);
    const long long P = (long long)a.N * a.Hu * a.SW;
    const int TU = a.pool ? G::T / 4 : G::T;
    a.tpp = (int)((P + TU - 1) / TU);
    const long long nblk = (long long)a.tpp * p.npan * a.NKT;
    const int nch = (a.C + G::CC - 1) / G::CC;
    a.parts = a.sums ? p.parts : 1;
    a.cpp = (nch + a.parts - 1) / a.parts;
    if (nblk <= 0 || nblk * a.parts > 0x7fffffffLL || nblk * a.parts * G::NTH > 0xffffffffLL) return hipErrorInvalidValue;
    a.nblk = (int)nblk;
    hipLaunchKernelGGL(split_kernel<G>, dim3((unsigned)(nblk * a.parts)), dim3(G::NTH), p.lds, st, a);
    if (a.parts > 1) {
        const dim3 grid((unsigned)(((long long)a.N * a.K * a.Hu * a.Wu + 255) / 256));
        if (a.pool) hipLaunchKernelGGL((parts_finish_kernel<G::R, true>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((parts_finish_kernel<G::R, false>), grid, dim3(256), 0, st, a);
    }
    return hipGetLastError();
}

template <int R, bool GEN> hipError_t launch_any(const SpArgs &a, const ContractPick &p, hipStream_t st)
{
    switch (p.cfg) {
    case 3: return launch_cfg<SpCfg<2, 2, 2, 4, R, GEN>>(a, p, st);
    case 4: return launch_cfg<SpCfg<2, 2, 2, 3, R, GEN>>(a, p, st);
    case 7: return launch_cfg<SpCfg<4, 2, 1, 2, R, GEN>>(a, p, st);
    case 8: return launch_cfg<SpCfg<2, 4, 1, 2, R, GEN>>(a, p, st);
    case 9: return launch_cfg<SpCfg<2, 4, 1, 1, R, GEN>>(a, p, st);
    }
    if constexpr (R == 3) {   // (for 5x5 the A operands of five taps leave no room for more accumulators)
        switch (p.cfg) {
        case 0: return launch_cfg<SpCfg<2, 2, 2, 7, R, GEN>>(a, p, st);
        case 1: return launch_cfg<SpCfg<2, 2, 2, 6, R, GEN>>(a, p, st);
        case 2: return launch_cfg<SpCfg<2, 2, 2, 5, R, GEN>>(a, p, st);
        case 5: return launch_cfg<SpCfg<4, 2, 1, 4, R, GEN>>(a, p, st);
        case 6: return launch_cfg<SpCfg<4, 2, 1, 3, R, GEN>>(a, p, st);
        }
    }
    return hipErrorInvalidValue;
}

}  // namespace

// The configuration of a launch, by a model of its time: rounds of work-groups over the 256 CUs, each taking per
// chunk its matrix instructions (32 clocks each on four SIMDs), the staging and a fixed part, then a first round
// trip to memory and its stores; matrix instructions and chunks take longer the fuller the chip is (it runs into its
// power limit: 2.4 GHz where few CUs work, 1.8 to 2.0 where all do).  Fitted to random geometries of the ranges that
// the contraction serves: 3x3 at strides 1 and 2, 31091 launches, standard deviation 6 %, its choice 0.8 % slower than
// the fastest one on average; 5x5, 4632, 5 %, 0.5 %.
struct SplitCost {
    double mfma, mfma_fill, stage, chunk, chunk_fill, round, store, launch;
};
constexpr SplitCost kSplitCost[] = {{0.916, 0.425, 53.1, 2077, 0.315, 7974, 1197, 2.28},    // 3x3
                                    {0.876, 0.325, 60.9, 3502, 0.805, 6873, 1215, 2.89}};   // 5x5
// With `divide`, launches that leave CUs idle may divide the input channels over up to kPartsMost work-groups per tile, where all of
// them still fit one round; the second launch, which adds up, costs 1.5 us and the sums' way (3 TB/s).  10 % stored, us gathered,
// contracted whole and divided, the estimate of the last: 512 -> 512 at 14x14, N = 1: 19.0, 27.4, 14.4 (15.2); at 7x7: 17.2, 26.4,
// 11.0 (11.2); 512 -> 128 at 20x20: 17.7, 26.6, 11.9 (11.9); 256 -> 256 at 28x28, where dividing gives little: 15.9, 16.2, 14.5.
constexpr int kPartsMost = 16;
constexpr long long kPartsBytes = 64LL << 20;
// The units of a call (see the top of this file)
struct Units {
    int IL, N, W, pw, Hu, Wu, xstep, ystep, rext;
    Units(int N_, int W_, int R, int Ho, int Wo, int sh, int sw, int pw_, bool in4, bool pool)
    {
        IL = in4 ? 4 : 1;
        N = in4 ? (N_ + 3) / 4 : N_; W = W_ * IL; pw = pw_ * IL;
        Hu = pool ? Ho / 2 : Ho; Wu = (pool ? Wo / 2 : Wo) * IL;
        xstep = pool ? 2 * sw : sw; ystep = pool ? 2 * sh : sh; rext = pool ? R + sh : R;
    }
};
ContractPick split_pick(int N, int C, int K, int H, int W, int R, int S, int Ho, int Wo, int sh, int sw, int pw, bool divide, bool in4, bool pool)
{
    ContractPick best;
    if (R != S || (R != 3 && R != 5) || (R == 5 && (in4 || pool)) || (pool && (Ho < 2 || Wo < 2)) || W > 0x10000000) return best;
    const Units u(N, W, R, Ho, Wo, sh, sw, pw, in4, pool);
    const int real = Ho * Wo;              // (results per image and channel)
    N = u.N; W = u.W; pw = u.pw; Ho = u.Hu; Wo = u.Wu;
    // (rows are loaded four columns at a time)
    if (W < 4) return best;
    // weights and the images a stripe can touch are addressed with 32-bit byte offsets, pixels of a
    // panel numbered with ints
    const long long big = 0x7fffffffLL;
    if (split_packed_bytes(K, C, R * S) >= big || (long long)N * Ho * (Wo + 64) >= big || (long long)N * H * W >= big ||
        (long long)N * ((long long)(Ho - 1) * u.ystep + u.rext) >= big || (Ho - 1) * (long long)u.ystep + u.rext > 40000 || Wo > 40000)
        return best;
    const SplitCost &m = kSplitCost[R == 3 ? 0 : 1];
    int last_npan = 0;
    for (int target : {40000, 64, 48, 32, 24, 16, 12, 8, 6}) {          // widths of a panel
        const int npan0 = (Wo + target - 1) / target, SW = ((Wo + npan0 - 1) / npan0 + u.IL - 1) / u.IL * u.IL, npan = (Wo + SW - 1) / SW;
        if (npan == last_npan) continue;
        last_npan = npan;
        const int pitch = (((pool ? 2 : 1) * SW / u.IL - 1) * sw + S) * u.IL;
        // columns of a panel that lie in the image: at least one load's worth, at most qpr
        int most = 0, least = W;
        for (int p = 0; p < npan; ++p) {
            const long long c0 = (long long)p * SW * u.xstep - pw, first = c0 > 0 ? c0 : 0, end = c0 + pitch < W ? c0 + pitch : W;
            const int have = end > first ? (int)(end - first) : 0;
            most = have > most ? have : most;
            least = have < least ? have : least;
        }
        if (least < 4) continue;
        const int qpr = (most + 3) / 4;
        const long long P = (long long)N * Ho * SW;
        for (int g = 0; g < kNGeo; ++g) {
            const Geo &q = kGeo[g];
            const int T = (pool ? 8 : 32) * q.NB, NT = (q.NB + q.NW - 1) / q.NW;
            if (R == 5 && NT > 2) continue;
            const int rows = (T + SW - 2) / SW + 1;             // rows of units a tile can touch
            const int cross = (rows - 1 + Ho - 1) / Ho;         // image boundaries among them
            const long long nrow = (long long)(rows - 1) * u.ystep + u.rext + (long long)cross * (R > sh ? R - sh : 0);
            if (nrow * qpr > 64 * 8 / (2 * q.KS)) continue;
            if ((cross + 2LL) * (C + 8) * H * W * 4 >= big - 64) continue;
            const long long npx = nrow * pitch;
            const long long buf = npx * 48 * 2 * q.KS;
            const long long red = 8LL * NT * 64 * 64;
            const long long lds = 2 * buf > red ? 2 * buf : red;
            if (lds > kLdsMax) continue;
            const long long nwg = (P + T - 1) / T * npan * ((K + 32 * q.MW - 1) / (32 * q.MW));
            const int nch = (C + 16 * q.KS - 1) / (16 * q.KS);
            const double mfma = 48.0 * q.MW * q.NB * q.KS * R * S;
            for (int parts = 1; parts <= nch; ++parts) {
                const int cpp = (nch + parts - 1) / parts;
                if ((parts - 1) * cpp >= nch) continue;         // (the last one would have none)
                const double sums = 4.0 * parts * N * u.IL * K * real;
                if (parts > 1 && (!divide || parts > kPartsMost || nwg * parts > 256 || sums > kPartsBytes)) break;
                const double groups = (double)nwg * parts, rounds = (double)((nwg * parts + 255) / 256), fill = groups / (256 * rounds);
                const double chunk = m.mfma * (1 + m.mfma_fill * fill) * mfma + m.stage * q.KS / 32 * (double)npx + m.chunk * (1 + m.chunk_fill * fill);
                double seconds = rounds * (cpp * chunk + m.round + m.store * q.MW * q.NB) / 2.4e9 + m.launch * 1e-6;
                if (parts > 1) seconds += 1.5e-6 + sums / 3e12;
                if (best.cfg < 0 || seconds < best.seconds) {
                    best.seconds = seconds;
                    best.cfg = g; best.npan = npan; best.lds = (int)lds; best.qpr = qpr;
                    best.SW = SW; best.pitch = pitch; best.PL = (int)npx; best.buf = (int)buf;
                    best.parts = parts;
                }
            }
        }
    }
    return best;
}

hipError_t launch_split_rows(const int *rowptr, const uint32_t *idx, const float *val, int K, int C, int RS, void *packed, hipStream_t st)
{
    const int nslice = (C + 15) / 16;
    const dim3 grid((unsigned)((long long)nslice * ((K + 31) / 32)));
    if (RS == 9) hipLaunchKernelGGL(split_rows_kernel<9>, grid, dim3(512), 0, st, rowptr, idx, val, K, nslice, static_cast<u4v *>(packed));
    else if (RS == 25) hipLaunchKernelGGL(split_rows_kernel<25>, grid, dim3(512), 0, st, rowptr, idx, val, K, nslice, static_cast<u4v *>(packed));
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_split_dense(const float *x, const void *packed, const int *rowptr, const uint32_t *idx, const float *val, int N, int C,
                              int H, int W, int K, int R, int Ho, int Wo, int sh, int sw, int ph, int pw, const float *bias, int act,
                              float *y, int in4, int out4, int pool, const ContractPick &p, float *sums, hipStream_t st)
{
    if (p.cfg < 0 || (out4 && !in4)) return hipErrorInvalidValue;
    SpArgs a = {};
    const Units u(N, W, R, Ho, Wo, sh, sw, pw, in4 != 0, pool != 0);
    a.sums = sums;
    a.x = x; a.w = static_cast<const char *>(packed); a.bias = bias; a.y = y;
    a.N = u.N; a.C = C; a.H = H; a.W = u.W; a.K = K; a.nslice = (C + 15) / 16; a.nkb = (K + 31) / 32;
    a.sh = sh; a.sw = sw; a.ph = ph; a.pw = u.pw; a.act = act;
    a.il = in4 ? 2 : 0; a.pool = pool; a.out4 = out4; a.images = N;
    a.Hu = u.Hu; a.Wu = u.Wu; a.ystep = u.ystep; a.rext = u.rext;
    a.slow.rowptr = rowptr; a.slow.idx = idx; a.slow.val = val;
    if (in4 || pool) return R == 3 ? launch_any<3, true>(a, p, st) : hipErrorInvalidValue;
    return R == 3 ? launch_any<3, false>(a, p, st) : launch_any<5, false>(a, p, st);
}

hipError_t launch_split_bank(const float *w, int K, int C, void *packed, hipStream_t st)
{
    const int nslice = (C + 15) / 16;
    hipLaunchKernelGGL(split_dense_kernel, dim3((unsigned)((long long)nslice * ((K + 31) / 32))), dim3(kBankThreads), 0, st, w, K, C, nslice,
                       static_cast<u4v *>(packed));
    return hipGetLastError();
}

hipError_t launch_split_input(const fscnn_input *in, const void *packed, const float *w, int wk, int wc, int wt, int K, int Ho, int Wo,
                              int ph, int pw, const float *bias, int relu, float *y, const ContractPick &p, const int *gate,
                              int gate_from, hipStream_t st)
{
    if (p.cfg < 0 || !in->dense) return hipErrorInvalidValue;
    SpArgs a = {};
    a.gate = gate; a.gate_from = gate_from; a.x = in->dense;
    a.w = static_cast<const char *>(packed); a.bias = bias; a.y = y;
    a.N = a.images = in->N; a.C = in->C; a.H = in->H; a.W = in->W; a.K = K; a.nslice = (in->C + 15) / 16; a.nkb = (K + 31) / 32;
    a.Hu = Ho; a.Wu = Wo; a.ystep = 1; a.rext = 3;
    a.sh = a.sw = 1; a.ph = ph; a.pw = pw; a.act = relu;
    a.slow.cptr = in->cptr; a.slow.cidx = in->cidx; a.slow.xval = in->xval; a.slow.NCP = in->NCH;
    a.slow.w = w; a.slow.wk = wk; a.slow.wc = wc; a.slow.wt = wt;
    return launch_any<3, false>(a, p, st);
}

}  // namespace fscnn
