// Host-side declarations shared by the NestedFP library's translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include <atomic>
#include <utility>

namespace nfp {

// status codes mirror include/nestedfp.h
enum { kOk = 0, kErrArg = 1, kErrShape = 2, kErrRange = 3, kErrWorkspace = 4, kErrHip = 5 };

inline int hip_ok(hipError_t e) { return e == hipSuccess ? kOk : kErrHip; }

// weight operand kinds of the GEMM kernels
//   kPlainF16      : FP16 weights, row-major [N,K] (row stride ldw)
//   kNestedF16     : the two byte planes in packed 1 KB blocks
//   kE4M3          : E4M3 bytes (the upper plane) in packed 1 KB blocks
//   kE4M3Quant, kE4M3QuantRow: as kE4M3, kE4M3Row, FP16 activations quantised per token inside the kernel
//   kNestedF16Row  : the two byte planes row-major [N,K], regrouped into operand order in flight
//   kE4M3Row       : E4M3 bytes row-major [N,K]
//   kPlainF16Packed: FP16 weights in packed 2 KB blocks (the like-for-like partner of kNestedF16)
enum WeightKind { kPlainF16 = 0, kNestedF16 = 1, kE4M3 = 2, kE4M3Quant = 3,
                  kNestedF16Row = 4, kE4M3Row = 5, kPlainF16Packed = 6, kE4M3QuantRow = 7, kNumKinds = 8 };

constexpr bool kind_quantizes(int k) { return k == kE4M3Quant || k == kE4M3QuantRow; }
constexpr bool kind_is_fp8(int k) { return k == kE4M3 || k == kE4M3Row || kind_quantizes(k); }
constexpr bool kind_is_nested(int k) { return k == kNestedF16 || k == kNestedF16Row; }
// weights stored in blocks of 16 rows x 64 columns, lane order inside
constexpr bool kind_is_packed(int k) { return k == kNestedF16 || k == kE4M3 || k == kE4M3Quant || k == kPlainF16Packed; }
// bytes of one weight in the array(s) the kernel reads
constexpr int kind_elem_bytes(int k) { return (k == kPlainF16 || k == kPlainF16Packed) ? 2 : 1; }
// which cost table / routing rule a kind follows: 0 plain FP16 through LDS, 1 FP16 operands through
// registers (both plane layouts, packed FP16), 2 E4M3
constexpr int kind_class(int k) { return k == kPlainF16 ? 0 : (kind_is_fp8(k) ? 2 : 1); }

// bytes of one weight array of an [N,K] layer as the kernels address it (plain row-major FP16:
// row stride ldw elements; row-major planes are dense; packed kinds are padded to whole blocks)
inline int64_t weight_array_bytes(int kind, int64_t N, int64_t K, int64_t ldw) {
    if (N <= 0) return 0;
    if (kind_is_packed(kind)) return ((N + 15) / 16 * 16) * ((K + 63) / 64 * 64) * kind_elem_bytes(kind);
    if (kind == kPlainF16) return (N - 1) * 2 * ldw + 2 * K;
    return N * K;
}

struct GemmArgs {
    // activations: fp16 X (kPlainF16 / kNestedF16) or E4M3 Xq with per-row scales (kE4M3)
    const void *X;        // uint16_t* or uint8_t*
    int64_t ldx;          // elements
    const float *scales;  // [M], kE4M3 only
    const float *static_scale;  // kE4M3Quant: optional per-tensor activation scale (device float)
    float w_scale;        // kE4M3 only
    // weights
    const void *W0;       // fp16 W, or upper plane, or E4M3 weights
    const void *W1;       // lower plane (kNestedF16 only)
    int64_t ldw;          // elements (plain fp16 only; planes are dense)
    int64_t M, N, K;
    uint16_t *Y;
    int64_t ldy;
    float *partials;      // split-K scratch (may be NULL if split == 1)
    size_t partial_bytes;
    uint32_t *counters;   // kMaxCounters arrival counters, all zero between calls (NULL: reduce in a second launch)
    bool bounded;         // K splits of more than 64 tokens that fit the fixed scratch only (see nestedfp_gemm_static)
};

// arrival counters at the start of every workspace: one per output tile of a split launch
constexpr int kMaxCounters = 4096;
constexpr size_t kCounterBytes = kMaxCounters * sizeof(uint32_t);

// tuning knobs (negative = built-in choice)
struct Tuning {
    int64_t small_max_m;     // largest M routed to the streaming kernel
    int64_t small_split;     // grid-level split-K of the streaming kernel
    int64_t small_spw;       // K-steps per wave (2, 4, or 8: row-major FP16 operands with a long K only)
    int64_t small_tiles;     // 16-row weight tiles per workgroup
    int64_t small_interleave;  // 1: a workgroup's tiles are strided by the grid size
    int64_t large_split;     // grid-level split-K of the tiled kernel
    int64_t large_bm;        // tokens per tile of the tiled kernel (64, 128 or 256)
    int64_t large_bn;        // weight rows per tile (128 or 256; unset: same as large_bm)
    int64_t small_fuse_quant;  // 1 / 0: quantise activations inside the streaming kernel wherever it can / nowhere
    int64_t quant_hw;        // 1: hardware E4M3 convert, 0: integer rounding
    int64_t large_xcd_map;   // 0: tiles in launch order instead of grouped by XCD (tiled kernels)
    int64_t fused_reduce;    // 0: split-K partials are summed by a second launch instead of the last workgroup
    int64_t large_deep;      // 1 / 0: force / forbid the deeper load pipelines of the tiled kernels (tiles below 256 x 256)
    int64_t large_height;    // height of token tiles of 256 where they exist cut down: 160, 192, 224 or 256
    int64_t large_rows;      // 1 / 0: row-major planes reach tiles above 64 tokens through LDS / straight into registers
    int64_t tuned_table;     // 0: the tiled kernels' launch shape always comes from the cost model, never from the table of timed shapes
    int64_t quant_onepass;   // 1 / 0: force / forbid the single-pass activation quantisation (rows kept in registers) where it fits
};
Tuning &tuning();
uint32_t tuning_epoch();                               // counts the changes of the knobs

// Launch shapes already worked out in this host thread, by problem: choosing one prices a hundred or so
// candidates (1-3 us of host time), and every call asks several times.  Keyed by sizes and a class of kinds
// alone; a fixed number of entries (20-40 KB), dropped when a knob changes.  512 entries in pairs hold the four
// linears of a layer in two modes at 64 batch sizes; with 64 single ones, batches of 1 ... 16 tokens in turn
// were worked out anew each time (workspace queries of 4.1 us on average against 0.5).
template <typename Config>
struct PlanCache {
    struct Entry {
        int64_t M, N, K;
        int cls;
        uint32_t epoch;
        bool set;
        Config config;
        bool is(int cls_, int64_t M_, int64_t N_, int64_t K_, uint32_t epoch_) const {
            return set && epoch == epoch_ && M == M_ && N == N_ && K == K_ && cls == cls_;
        }
    };
    Entry entries[256][2] = {};
    template <typename Choose>
    const Config &get(int cls, int64_t M, int64_t N, int64_t K, Choose choose) {
        const uint64_t h = ((uint64_t)M * 0x9e3779b97f4a7c15ull) ^ ((uint64_t)N * 0xc2b2ae3d27d4eb4full) ^
                           ((uint64_t)K * 0x165667b19e3779f9ull) ^ (uint64_t)cls * 0x27d4eb2f165667c5ull;
        Entry *e = entries[h >> 56];
        const uint32_t epoch = tuning_epoch();
        if (e[0].is(cls, M, N, K, epoch)) return e[0].config;
        if (!e[1].is(cls, M, N, K, epoch)) e[1] = {M, N, K, cls, epoch, true, choose()};
        std::swap(e[0], e[1]);                                 // the entry used last is kept longest
        return e[0].config;
    }
};

int launch_decompose(const uint16_t *W, int64_t N, int64_t K, int64_t ldw, uint8_t *upper,
                     uint8_t *lower, uint64_t *counter, bool clear, bool packed, hipStream_t stream);      // clear: the counter starts at zero
int launch_range_check(const uint16_t *W, int64_t N, int64_t K, int64_t ldw, uint64_t *counter, bool clear,
                       hipStream_t stream);
int launch_hand_on_count(uint64_t *counter, uint64_t *dev, uint64_t *host, hipStream_t stream);
int launch_zero_u64(uint64_t *p, hipStream_t stream);
int launch_reconstruct(const uint8_t *upper, const uint8_t *lower, int64_t N, int64_t K,
                       uint16_t *W, int64_t ldw, bool packed, hipStream_t stream);
int launch_pack_fp16(const uint16_t *W, int64_t N, int64_t K, int64_t ldw, uint8_t *dst, hipStream_t stream);
int launch_zero_words(uint32_t *p, int n, hipStream_t stream);
size_t plane_bytes(int64_t N, int64_t K);
int launch_pack_plane(const uint8_t *src, int64_t N, int64_t K, int64_t ld, uint8_t *dst, hipStream_t stream);
int launch_unpack_plane(const uint8_t *src, int64_t N, int64_t K, uint8_t *dst, int64_t ld, hipStream_t stream);
int launch_quantize_act(const uint16_t *X, int64_t M, int64_t K, int64_t ldx,
                        const float *static_scale, uint8_t *Xq, int64_t ldq, float *scales, hipStream_t stream);

// streaming (small-M) and tiled (large-M) GEMM families
bool small_gemm_supports(int kind, int64_t M, int64_t N, int64_t K, int64_t ldw);
double small_gemm_cost(int kind, int64_t M, int64_t N, int64_t K);     // priced microseconds of the chosen launch shape
struct Tile64Plan { double cost; int split; };
Tile64Plan tile64_plan(int kind, int64_t M, int64_t N, int64_t K);     // the same for the 64-token tiles, and their K split
bool small_gemm_fuses_quant(int64_t M, int64_t N, int64_t K);
size_t small_gemm_partial_bytes(int kind, int64_t M, int64_t N, int64_t K);
int launch_small_gemm(int kind, const GemmArgs &a, hipStream_t stream);
bool rows_by_pairs(int tm, int64_t M, int64_t N, int64_t K, int64_t row_bytes, int split);   // row-major planes, 64-token tiles and the deeper pipeline
bool rows_through_lds(int tm, int tn, int64_t M, int64_t K, int64_t row_bytes, int split);           // the other tiles
size_t large_gemm_partial_bytes(int kind, int64_t M, int64_t N, int64_t K);
size_t large_gemm_bounded_bytes(int kind, int64_t M, int64_t N, int64_t K);      // with GemmArgs::bounded
int large_gemm_height(int kind, int64_t M, int64_t N, int64_t K);                // tokens per tile
int launch_large_gemm(int kind, const GemmArgs &a, hipStream_t stream);

// Row stride of the split-K partial sums [slice][token][ld]: whole groups of four columns, so that they are
// written and read 16 bytes per lane whatever N is (with N itself, odd layers paid four narrow accesses
// each: (2903, 9168) in FP16 mode at 40 tokens 29.6 us against 21).
constexpr int64_t partial_ld(int64_t N) { return (N + 3) & ~(int64_t)3; }

// Workspace layout: [arrival counters : kCounterBytes][Xq : M rows of K bytes, or of xq_row(K) where there is room][scales :
// M floats][split-K partials], each part rounded up to 256 bytes; 0 if nothing but the counters would be in it.  What follows
// is the least, with dense rows.
constexpr size_t round256(size_t b) { return (b + 255) & ~(size_t)255; }
constexpr size_t workspace_need(size_t partial_bytes, int64_t M, int64_t K, bool quantize) {
    const size_t b = round256(partial_bytes) +
                     (quantize ? round256((size_t)M * (size_t)K) + round256((size_t)M * sizeof(float)) : 0);
    return b > 0 ? b + kCounterBytes : 0;
}

// Rows of the quantised activations in a workspace start on 128-byte lines where there is room: the tiled kernels copy 128 bytes of
// 8 rows per instruction, which are 8 lines then and 16 otherwise.  FP8 mode on 17 layers with K % 128 != 0, time without / with, geometric
// mean: 16 tokens 1.02, 64 tokens 1.07, 200 tokens 1.05, 589 tokens 1.08, 1024 tokens 1.10, 5000 tokens 1.05; (24434, 4064) at 1024 tokens 138.5 / 115.1
// us, (7600, 7600) 77.8 / 67.3; none slower by more than the timings differ.
// Queries ask for that room unless it would push them past the fixed scratch below, calls do without it.
constexpr int64_t xq_row(int64_t K) { return (K + 127) & ~(int64_t)127; }
constexpr size_t xq_padding(int64_t M, int64_t K) { return round256((size_t)M * (size_t)xq_row(K)) - round256((size_t)M * (size_t)K); }

// The entry point without a workspace argument has a fixed scratch, and takes every problem that fits it.
constexpr size_t kStaticScratch = (size_t)32 << 20;
constexpr bool static_scratch_holds(int split, int64_t M, int64_t N, int64_t K, bool quantize, int64_t ld) {
    return workspace_need(split > 1 ? (size_t)split * (size_t)M * (size_t)ld * sizeof(float) : 0, M, K, quantize) <= kStaticScratch;
}
// A split that only the padding of the rows would push past that scratch is not taken -- by any entry point, so
// that all of them give the same bits: (1221, 167, 22112) in FP8 mode needs 33545472 bytes in three slices
// unpadded, 33584384 padded.
constexpr bool padded_split_fits(int split, int64_t M, int64_t N, int64_t K, bool quantize) {
    return static_scratch_holds(split, M, N, K, quantize, partial_ld(N)) || !static_scratch_holds(split, M, N, K, quantize, N);
}

int launch_splitk_reduce(const float *partials, int S, int64_t M, int64_t N, const float *scales,
                         float w_scale, uint16_t *Y, int64_t ldy, hipStream_t stream);

bool large_gemm_supports(int kind, int64_t K, int64_t ldx, int64_t ldw);
int launch_probe_stream_read(const void *src, size_t bytes, uint32_t *sink, hipStream_t stream);
int launch_probe_stream_read_sparse(const void *src, size_t bytes, uint32_t *sink, hipStream_t stream);
int launch_probe_mfma(const void *operands, int fp8, int iters, uint32_t *sink, double *flops_host,
                      hipStream_t stream);

bool use_small_gemm(int64_t M);
bool route_small(int kind, int64_t M, int64_t N, int64_t K, int64_t ldw);     // which of the two families a problem runs on

}  // namespace nfp
