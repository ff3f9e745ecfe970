// Internal declarations shared by the translation units of libfscnn.so.
// Nothing here is part of the C ABI (see include/fscnn.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <mutex>
#include <vector>

#include "fscnn.h"

namespace fscnn {

constexpr uint64_t kFilterMagic = 0x4653434e4e464c54ull;  // "FSCNNFLT"
constexpr uint64_t kInputMagic = 0x4653434e4e494e50ull;   // "FSCNNINP"
constexpr uint64_t kDenseMagic = 0x4653434e4e44454eull;   // "FSCNNDEN"

// One nonzero as the convolution kernel streams it: the byte offset of the tap
// (c mod CC, r, s) inside the LDS input tile, and the weight (the paper's node
// {index, value}, Sec. 3, with the index pre-multiplied for the tile geometry).
struct Rec {
    uint32_t off;
    float val;
};

// Geometry of one kernel configuration of the tiled sparse-filter convolution.
struct SfGeom {
    int BV, LW, LHR, NV, SLOTS, WAVES, CC;  // template parameters
    int R, S;                               // filter extent the instance is built for
    int TH, TW, IMGS;                       // output tile and images per work-group
    int IN_ROWS, PITCH;                     // LDS rows per channel, BV-vectors per row
    int KG;                                 // output channels per work-group
    int STRIDE;                             // stride (both axes) the instance is built for
    int DENSE;                              // 1: the plan lists every tap of every chunk, SLOTS weights per tap
    int SPLIT;                              // 1: built with the channel split
    int REGST;                              // 1: NCHW input staged through registers
    int lds_bytes;
};

// Activation code carried by the kernels' `relu` argument: 0 = none, 1 = ReLU, anything else =
// the bit pattern of a LeakyReLU slope (y > 0 ? y : slope * y).  A slope whose bits are 0 or 1
// (0.0f, the smallest denormal) is ReLU to rounding and is mapped to 1 by act_code().
__host__ __device__ inline float act_apply(float r, int act)
{
    // none / ReLU first (the common cases: one compare-and-select); the LeakyReLU fix-up sits
    // behind a branch on the wave-uniform code so that the other two do not pay for it
    float y = act == 1 ? (r > 0.0f ? r : 0.0f) : r;
    if (__builtin_expect((act & ~1) != 0, 0)) {
        union { int i; float f; } u;
        u.i = act;
        y = r > 0.0f ? r : r * u.f;
    }
    return y;
}
inline int act_code(float negative_slope)
{
    union { int i; float f; } u;
    u.f = negative_slope;
    return (u.i == 0 || u.i == 1) ? 1 : u.i;
}

constexpr int kPlanSpare = 12;  // zero records appended to a plan's stream (reader prefetch)

struct SfPlan {
    int variant = 0;   // 1-based index into the variant table
    bool direct = false;
    SfGeom g{};
    int NCH = 0, NG = 0;
    long long nrec = 0;       // records (= nonzeros); the array carries kPlanSpare spare entries
    int *segptr = nullptr;    // [NG*NCH*KG + 1], bucket order (group, wave, chunk, slot); behind the records
    Rec *recs = nullptr;      // [nrec + kPlanSpare]; owns the allocation
    // Scratch of the channel-split mode (small problems): one buffer per stream that has used the
    // plan in that mode, so that calls on different streams never share one.  Grown on demand.
    struct SplitScratch {
        hipStream_t stream;
        float *buf;
        size_t bytes;
    };
    std::vector<SplitScratch> split, outgrown;
    size_t recs_bytes = 0, packed_bytes = 0, parts_bytes = 0;   // of the allocations
    // The plan of the contraction on the matrix cores (variant kContractPlan): the bank as a dense
    // packed array (contract_packed_index), zeros where nothing is stored; behind it an int that is
    // non-zero if a stored value is Inf or NaN (16 bytes).
    float *packed = nullptr;
    // The plan of the contraction in bfloat16 parts (variant kSplitPlan): the parts (split_packed_bytes).
    void *parts = nullptr;
};
constexpr int kDirectPlan = -1, kContractPlan = -2, kSplitPlan = -3;

// How a call of the contraction on the matrix cores would be launched (cfg < 0: it is not served) and an estimate of its time.  Host only.
struct ContractPick {
    int cfg = -1, npan = 1, lds = 0, SW = 0, pitch = 0, PL = 0, buf = 0;
    int qpr = 0;                           // in bfloat16 parts: loads of four columns per row of a stripe
    int parts = 1;                         // likewise: work-groups that the input channels of a tile are divided over
    double seconds = 0;
};

// How a sparse-filter call is served.
struct SfRoute {
    int key[9];
    int variant = 0;                       // configuration, or kDirectPlan
    int band_shift = 0, band_h = 0;        // sf_choose_bands
    int csplit = 1;                        // sf_choose_csplit
    bool contract = false;                 // by the contraction, as `pick` says, once its plan is there
    ContractPick pick;
    bool split = false;                    // by the contraction in bfloat16 parts, as `spick` says, once its plan is there
    ContractPick spick;
    bool pointwise = false;                // by the kernel for 1x1 filters
};

struct SiGeom {
    int CC;  // channels per chunk of the compressed activation's chunk pointers
};
hipError_t launch_dense_transpose(const float *w, int K, int C, int RS, int Kpad, float *wT,
                                  hipStream_t st);
int si_variant_count();
hipError_t launch_conv_si_prepared(const fscnn_input *in, const fscnn_dense *d, int Ho, int Wo, int ph,
                                   int pw, const float *bias, int relu, float *y, int variant,
                                   hipStream_t st);

}  // namespace fscnn

struct fscnn_filter {
    uint64_t magic;
    int device;
    int K, C, R, S;
    long long nnz;
    int *rowptr;    // device [K+1], `fewest` behind them; owns an allocation
    uint32_t *idx;  // device [nnz]; owns an allocation
    float *val;     // device [nnz], behind the indices
    int fewest = 0;                           // stored values of the filter that stores the fewest, of those that store any
    size_t rowptr_bytes = 0, idx_bytes = 0;   // of the allocations
    std::atomic<bool> in_order{true};         // no call has used the handle on another stream than the default one
    std::mutex mu;
    std::mutex launching;                     // held over the launches of a call that share scratch (taken before mu)
    std::vector<fscnn::SfPlan *> plans;
    // how automatic calls of a geometry are served (route_call in api.hip): the last few geometries asked for
    std::vector<fscnn::SfRoute> routes;
    size_t next_route = 0;
};

struct fscnn_input {
    uint64_t magic;
    int device;
    int N, C, H, W;
    long long nnz;   // -1: not fetched yet (the handle was filled without a host synchronisation;
                     // input_nnz() waits for `filled` and reads cptr's last element)
    int CC, NCH;     // chunking of the channel axis used by cptr
    uint32_t *cidx;  // device [nnz]
    float *xval;     // device [nnz]
    int *cptr;       // device [N*H*W*NCH + 1]: cptr[p*NCH + j] = first entry of pixel p with
                     // c >= j*CC; pixel p's row is [cptr[p*NCH], cptr[(p+1)*NCH])
    // device N x C x H x W: the activation as it was, where the handle keeps it (below).  Every pass that writes the lists renews it as
    // well, in device order: a captured pass or a captured reader may meet the handle after any other fill
    const float *dense = nullptr;
    // the device allocations behind the arrays: pointers (and the scratch they are made from), then
    // indices and values (null where they are part of the first: small or emitted activations)
    void *ptr_block, *node_block;
    size_t ptr_bytes = 0, node_bytes = 0;
    mutable std::atomic<bool> in_order{true};   // no call has used the handle on another stream than the default one
    long long unused = 0;   // bytes of indices and values allocated ahead and not stored
    // a handle made by an emitting convolution has ONE allocation (ptr_block) of emit_bytes, sized
    // for the worst case, with room for the dense result iff emit_has_y; 0 for other handles
    size_t emit_bytes = 0;
    bool emit_has_y = false;
    // room for the caller's bank in bfloat16 parts, one buffer per stream and capture that has needed it (bank_scratch in api.hip)
    struct Bank {
        hipStream_t stream;
        void *buf;
        size_t bytes;
        unsigned long long graph;   // the capture that has it; 0: none
    };
    mutable std::mutex mu;   // held over the launches that write and read such room
    mutable std::vector<Bank> banks;
    // the pass that fills the handle runs on `made_on` and may still be in flight when the
    // handle is returned; `filled` is recorded behind it, for users on other streams
    hipStream_t made_on;
    hipEvent_t filled;
};

// Dense filter bank prepared for the sparse-input convolution: a K-contiguous copy
// wT[c][r][s][k] (k padded to Kpad with zeros), built once.
struct fscnn_dense {
    uint64_t magic;
    int device;
    int K, C, R, S, Kpad;
    float *wT;       // device [C*R*S*Kpad]; the arrays below follow it in the same allocation
    float *packed;   // 3x3: the bank in the order of the contraction's A operands; else, or where there was no room for it, NULL
    void *parts;     // likewise, in bfloat16 parts (split_packed_bytes)
    int *flag;       // 3x3: non-zero if the bank holds an Inf or NaN
};

namespace fscnn {

// ---- compress.hip
// cnt: K + scan_tmp_elems(K) ints; rowptr: K + 2, the last one for the stored values of the filter that stores the fewest, of those that store
// any (INT_MAX: none does).  slot: HostWord::slot() of the word `host`, which receives the number of stored values, and that one behind it
hipError_t launch_filter_count(const float *w, int K, long long row, int *cnt, int *rowptr, int slot, int *host, hipStream_t st);
// out[0..n] = exclusive scan of in[0..n-1] (out[n] = total); tmp: scan_tmp_elems(n) ints of scratch; host: receives the total as
// well (pinned memory), or NULL.  fewest: out[n + 1] and the int behind *host receive the smallest of in[] above 0 (INT_MAX: none is)
long long scan_tmp_elems(long long n);
hipError_t launch_exclusive_scan(const int *in, int *out, long long n, int *tmp, int *host, bool fewest, hipStream_t st);
// slot, host: of a word that receives 0 when idx and val are there for every stream; -1: none does
hipError_t launch_filter_pack(const float *w, int K, long long row, const int *rowptr,
                              uint32_t *idx, float *val, int slot, int *host, hipStream_t st);
// pointers and records; recs NULL: the pointers alone, and no word.  scratch: plan_scratch_elems() ints; slot, host: as above
long long plan_scratch_elems(const SfGeom &g, int NCH, int NG);
hipError_t launch_plan(const int *rowptr, const uint32_t *idx, const float *val, int K, int R, int S, const SfGeom &g, int NCH, int NG,
                       int *scratch, int *segptr, Rec *recs, int slot, int *host, hipStream_t st);
// the taps-outer plan (SfGeom::DENSE): nrec = NG*WAVES*NCH*CC*R*S*SLOTS records plus the spare ones
hipError_t launch_plan_fill_dense(const int *rowptr, const uint32_t *idx, const float *val, int K, int C,
                                  int R, int S, const SfGeom &g, int NCH, int NG, long long nrec, Rec *recs,
                                  hipStream_t st);
// Activation compression: launch_input_sums adds up the stored values of every group of input_pixels(NCH) pixels, with cnt the counts
// per (pixel, step) instead of x; launch_input_fill then writes pointers and lists, and zeroes the `spare` entries that follow the last
// stored one.  scan: launch_input_sums scans the sums as well, which it has to where input_scans().  The number of stored values is then
// in scratch[input_groups] and in *host (pinned memory, or NULL) behind it, else behind launch_input_fill.
bool input_scans(long long npix, int NCH);
long long input_groups(long long npix, int NCH);
long long input_scratch_elems(long long npix, int NCH);   // ints
hipError_t launch_input_sums(const float *x, const int *cnt, int N, int C, int H, int W, int NCH, int *scratch, bool scan,
                             int *host, hipStream_t st);
// dense, if not NULL: receives x as well where dense_from values and more are stored
hipError_t launch_input_fill(const float *x, int N, int C, int H, int W, int NCH, int *scratch, bool scanned, int *cptr,
                             uint32_t *cidx, float *xval, int spare, float *dense, long long dense_from, int *host, hipStream_t st);
// An activation that stores a thirty-second of its values is kept dense as well: from there on a contraction may serve it
// (512 -> 512 at 28x28, N = 8: 132 us contracted, 157 gathered at 3 % stored)
inline long long input_dense_from(long long npix, int C) { return (npix * C + 31) / 32; }
hipError_t launch_maxpool2x2(const float *x, int N, int C, int H, int W, float *y, int n4,
                             hipStream_t st);
hipError_t launch_layout_convert(const float *src, int N, int C, int H, int W, int src_n4, float *dst,
                                 hipStream_t st);

// ---- conv_sf.hip
int sf_variant_count();
const char *sf_variant_name(int variant);
// false if the variant cannot serve RxS filters at this stride
bool sf_variant_geom(int variant, int R, int S, int sh, int sw, SfGeom *g);
int sf_choose_variant(int N, int C, int K, int H, int W, int R, int S, int stride, bool pool, bool n4,
                      double density, bool banded = false, bool emit = false);
bool sf_variant_has_layout(int variant, int in4, int out4, int pool);
// csplit > 1: scratch of the launch (N and Ho: slots and rows per band, where the image is banded), and
// the launch that clears its counters when it is new (a launch leaves them clear)
size_t sf_split_bytes(const SfGeom &g, int csplit, int N, int K, int Ho, int Wo);
constexpr int kSplitGroups = 256;   // (tile, channel group) pairs of a split launch, at most
hipError_t launch_split_clear(void *scratch, hipStream_t st);
// emit_cnt != nullptr (NCHW output, no pool only): the epilogue also stores, per output
// pixel p = (n*Ho + oy)*Wo + ox and step j of 8 output channels, the number of non-zero results into
// emit_cnt[p * ceil(K/8) + j] -- the counts the activation compressor scans
hipError_t launch_conv_sf_tiled(const SfPlan &p, const float *x, int N, int C, int H, int W, int K,
                                int Ho, int Wo, int ph, int pw, const float *bias, int relu,
                                float *y, int in4, int out4, int pool, int csplit, void *scratch,
                                int *emit_cnt, int band_shift, int band_h, hipStream_t st);
// band_shift, band_h of a launch: 4 / N bands of band_h output rows per image where a four-image
// configuration serves one or two images through NCHW tensors (then the work-groups of the launch,
// and with them the channel split, go by N << band_shift slots of band_h rows); else 0 and Ho
void sf_choose_bands(int variant, int N, int Ho, bool n4, bool pool, int *band_shift, int *band_h);
// 1, or the number of parts the input-channel range is split into for a small problem; the estimated time of that
// launch; emit: with emit_cnt below
int sf_choose_csplit(int variant, int N, int C, int K, int Ho, int Wo, double density, int in4, bool emit, double *us);
double sf_direct_us(int N, int K, int Ho, int Wo, long long nnz);   // the direct kernel's
hipError_t launch_conv_sf_direct(const int *rowptr, const uint32_t *idx, const float *val,
                                 const float *x, int N, int C, int H, int W, int K, int R, int S,
                                 int Ho, int Wo, int sh, int sw, int ph, int pw, const float *bias,
                                 int relu, float *y, hipStream_t st);

// ---- pointwise.hip: 1x1 filters at stride 1 without padding, both tensors NCHW or both N4; no plan
bool pointwise_serves(int N, int C, int H, int W, int K, bool n4);
double pointwise_us(int N, int C, int H, int W, int K, bool n4, long long nnz);   // estimated time
hipError_t launch_pointwise(const int *rowptr, const uint32_t *idx, const float *val, const float *x, int N, int C, int H, int W, int K,
                            bool n4, const float *bias, int act, float *y, hipStream_t st);
// ---- contract.hip: convolution as a dense contraction on the matrix cores
// (sources and banks: dense tensor; lists with a packed bank; lists with a K x C x 3 x 3 bank)
enum ContractForm { kContractDense, kContractLists, kContractListsRows };
ContractPick contract_pick(ContractForm form, int N, int C, int K, int H, int W, int R, int S, int Ho, int Wo, int sh, int sw);
// Packed banks: position of w[k][c][tap], and the number of floats (rows padded to 64 by zeros)
__host__ __device__ inline long long contract_packed_index(int k, int c, int rs, int RS, int nslice)
{
    return (((long long)(k >> 4) * nslice + (c >> 4)) * RS + rs) * 256 + ((c >> 2) & 3) * 64 + (k & 15) * 4 + (c & 3);
}
// (without the flag that follows a compressed bank's copy)
inline long long contract_packed_elems(int K, int C, int RS)
{
    return (long long)((K + 63) / 64 * 4) * ((C + 15) / 16) * RS * 256;
}
hipError_t launch_pack_rows(const int *rowptr, const uint32_t *idx, const float *val, int K, int C, int RS,
                            float *packed, hipStream_t st);
// both copies of a dense K x C x 3 x 3 bank (Kpad a multiple of 64) and its non-finite flag (16 bytes are cleared)
hipError_t launch_pack_dense(const float *w, int K, int C, int Kpad, float *packed, float *wT, int *flag, hipStream_t st);
// wflag: the packed bank's flag, if it is set every output is made entry by entry; NULL: not looked at
hipError_t launch_contract_dense(const float *x, const float *packed, const int *wflag, const int *rowptr, const uint32_t *idx,
                                 const float *val, int N, int C, int H, int W, int K, int R, int S, int Ho, int Wo,
                                 int sh, int sw, int ph, int pw, const float *bias, int act, float *y,
                                 const ContractPick &p, hipStream_t st);
// ---- contract_split.hip: the same contraction with the operands taken apart into three bfloat16 parts; 3x3 and 5x5
ContractPick split_pick(int N, int C, int K, int H, int W, int R, int S, int Ho, int Wo, int sh, int sw, int pw, bool divide, bool in4 = false,
                        bool pool = false);
// Packed banks, 16-bit words: [32 rows][16 channels][tap][part][octet of channels][row][channel]; the number of bytes
inline long long split_packed_bytes(int K, int C, int RS) { return (long long)((K + 31) / 32) * ((C + 15) / 16) * RS * 3072; }
hipError_t launch_split_rows(const int *rowptr, const uint32_t *idx, const float *val, int K, int C, int RS, void *packed, hipStream_t st);
// sums: room for the sums of p.parts parts (split_sums_bytes); NULL: one work-group per tile takes all channels
inline size_t split_sums_bytes(const ContractPick &p, int N, int K, int Ho, int Wo, bool in4)
{
    return 1024 + 4 * (size_t)p.parts * (in4 ? (N + 3) / 4 * 4 : N) * K * Ho * Wo;
}
hipError_t launch_split_dense(const float *x, const void *packed, const int *rowptr, const uint32_t *idx, const float *val, int N, int C,
                              int H, int W, int K, int R, int Ho, int Wo, int sh, int sw, int ph, int pw, const float *bias, int act,
                              float *y, int in4, int out4, int pool, const ContractPick &p, float *sums, hipStream_t st);
// the same parts of a dense K x C x 3 x 3 bank, and the convolution of a compressed activation with them; w[k*wk + c*wc + tap*wt]: the bank
// itself.  gate (device) with fewer than gate_from: the launch does nothing; NULL: it runs
hipError_t launch_split_bank(const float *w, int K, int C, void *packed, hipStream_t st);
hipError_t launch_split_input(const fscnn_input *in, const void *packed, const float *w, int wk, int wc, int wt, int K, int Ho, int Wo,
                              int ph, int pw, const float *bias, int relu, float *y, const ContractPick &p, const int *gate,
                              int gate_from, hipStream_t st);
// compressed activation, 3x3 at stride 1; with wflag: w is packed and wflag its non-finite flag,
// without: w is K x C x 3 x 3.  gate (device) with fewer than gate_from, or gate_to and more: the launch does nothing; NULL: it runs
hipError_t launch_contract_lists(const fscnn_input *in, const float *w, const int *wflag, int K, int Ho,
                                 int Wo, int ph, int pw, const float *bias, int relu, float *y,
                                 const ContractPick &p, const int *gate, int gate_from, int gate_to, hipStream_t st);
// How a sparse-input call (3x3, stride 1) is served: by the contraction in bfloat16 parts from split_from stored values
// on, else by the one in fp32 from `from` on
struct SiChoice {
    ContractPick pick, spick;
    long long from = 0, split_from = 0;
    int variant = 1;   // prepared banks: the gather configuration below
};
SiChoice si_choose(int N, int C, int H, int W, int K, int Ho, int Wo, int pw, bool prepared);

// ---- transpose.hip
long long reorder_workspace_bytes(long long n_buckets, long long nnz);  // -1: too large
// Size of the per-GPU static scratch of fscnn_sparse_transpose_noalloc, and its device address on
// the current GPU (looked up once per device).
constexpr long long kStaticScratchBytes = 8LL << 20;
hipError_t static_scratch(void **ptr);
hipError_t launch_reorder(bool tensor, const int *rowptr, const uint32_t *idx, const float *val,
                          int n_rows, int n_cols, int H, long long n_buckets, long long nnz,
                          int *tptr, uint32_t *tidx, float *tval, void *workspace, hipStream_t st);

// ---- conv_si.hip
constexpr int kSiCC = 8;   // channels per step of the compressed activation's chunk pointers
constexpr int kSiSpare = 8;  // entries allocated past the last (channel, value) pair (reader prefetch)
bool si_tiled_supported(int K, int C, int R, int S, int sh, int sw);
// c: how the contractions may serve the call (si_choose; NULL: they do not); bank: room for the bank in bfloat16 parts
// (split_packed_bytes), or NULL
hipError_t launch_conv_si(const fscnn_input *in, const float *w, int K, int R, int S, int Ho, int Wo,
                          int sh, int sw, int ph, int pw, const float *bias, int relu, float *y,
                          const SiChoice *c, void *bank, hipStream_t st);

}  // namespace fscnn
