// Streaming GEMM for decode-sized batches (M <= 64): Y = X * W^T with the weight stream
// read exactly once from HBM.  No weight is used by two waves, so nothing is staged for sharing; row-major
// weights and the activations pass through 2 KB of LDS per wave on their way into operand order.
// The paper's sweep starts at M = 32 with T_m >= 16 (Sec. 5.2, App. C); below that the
// linear layer is bound by HBM bandwidth, so the kernel is built around 128-bit loads of
// the byte planes with many loads in flight, K split across the waves of a workgroup,
// activations held in registers, and a fixed-order reduction.
//
// Weight rows are the MFMA "A" operand (lane l: row l%16 of a 16-row tile, K-group l/16),
// tokens (MT tiles of 16) the "B" operand, so each lane ends up with 4 consecutive output
// columns of one token: 8-byte stores of fp16.
//   plain FP16 : lane loads 32 B of FP16 weights              -> 2 x v_mfma_f32_16x16x32_f16
//   NestedFP16 : lane loads 16 B upper + 16 B lower, merges them (Sec. 4.2, Alg. 1) -> same
//   E4M3       : lane loads 2 x 16 B of E4M3 bytes (upper plane) -> 1 x v_mfma_f32_16x16x128_f8f6f4
// Every kind exists for two storage orders of the weights: row-major [N,K] (the two byte tensors
// of Sec. 4 "Overview" as they are, fetched in 128-byte pieces of 8 rows and regrouped through LDS) and
// packed blocks of 16 rows x 64 columns whose chunk order is the lane order, so that every load of a
// wave is one contiguous kilobyte.
// Columns past K and rows past N are never multiplied: their loads are sent out of the buffer's
// range and return zero, whatever the memory behind them holds.
#include <algorithm>
#include <cmath>

#include <type_traits>

#include "nfp_device.h"
#include "nfp_host.h"

namespace nfp {

struct SmallParams {
    const uint8_t *X;       // fp16 X (as bytes) or E4M3 Xq
    int64_t x_row_bytes;    // row stride of X in bytes
    const float *scales;    // [M] (kE4M3) or NULL
    const float *static_scale;  // kE4M3Quant: per-tensor activation scale or NULL (per token)
    int quant_hw;           // kE4M3Quant: hardware or integer E4M3 encoder
    float w_scale;
    const uint8_t *W0;      // fp16 W (bytes) / upper plane / E4M3 weights
    const uint8_t *W1;      // lower plane
    uint32_t w_row_bytes;   // row-major kinds: row stride of W0 (and W1) in bytes
    uint32_t tile_bytes;    // distance between consecutive 16-row tiles in bytes
    uint32_t w_bytes;       // addressable bytes of W0 (and W1), < 2^31
    int M, N, K;
    uint16_t *Y;
    int64_t ldy;
    float *partials;        // [S][M][ldp] when S > 1
    int ldp;                // see partial_ld
    uint32_t *counters;     // one arrival counter per workgroup column (zero between launches), or NULL
    int k_passes;           // K slices each wave walks through in turn
    int tiles_per_wg;       // 16-row weight tiles each workgroup walks through
    int tile_stride;        // distance between a workgroup's consecutive tiles (1 or gridDim.x)
    int rotate;             // 1: the waves' K-slices are rotated from workgroup to workgroup
    int vec_store;          // 1: 8-byte fp16 stores allowed
};

template <int KIND> struct StepK { static constexpr int value = kind_is_fp8(KIND) ? 128 : 64; };

// One K-step of weights for one 16-row tile, as loaded (32 bytes per lane).
struct WItem { u32x4 a, b; };   // plain: 32 B fp16; nested: upper, lower; e4m3: 32 B

// Buffer resource over a weight array: raw (unstructured) addressing with a byte range
// check, so reads past the end (N tail, look-ahead past the last tile) return zero
// without touching memory.  The arrays are smaller than 2 GiB (checked on the host), so an
// offset with bit 31 set is out of range by construction.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t weight_rsrc(const uint8_t *base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(base), 0, bytes, 0x00020000);
}

constexpr uint32_t kDead = 0x80000000u;               // an offset no weight array reaches

// Where the weights of a K-step sit.
// Packed kinds: lane l takes chunk l of a block, which is its MFMA operand; `voff` = lane part + tile
// part + the wave's slice; step S adds an immediate.
// Row-major kinds are fetched in pieces of 16 rows x 128 bytes by two instructions of 8 rows x 128
// bytes (lane l: row l / 8 of the eight, 16-byte chunk l % 8) and brought into operand order (lane l:
// row l % 16) through two kilobytes of LDS per wave, see Regroup.  Fetched in operand order instead
// -- 16 rows x 64 bytes per instruction -- every line is touched by two instructions, far enough apart
// to be requested twice, and non-temporal loads, which would keep the stream out of L2, cost a second
// trip to memory: a load-only kernel with the shape of this one reads (28672, 4096) in 47.8 us so, in
// 35.0 us by whole lines with the skew of the K-slices (see the kernel), and in 35.4 us from packed planes.
template <int KIND> struct WLayout {
    static constexpr bool PACKED = kind_is_packed(KIND);
    static constexpr int EB = kind_elem_bytes(KIND);
    static constexpr int KSTEP = StepK<KIND>::value;
    // bytes between consecutive K-steps of one tile
    static constexpr int STEP = (KSTEP / 64) * 1024 * EB;
    // packed: the second 16 bytes of a lane's step, relative to the first (NestedFP: the other plane, same offset)
    static constexpr int SECOND = kind_is_nested(KIND) ? 0 : 1024;
};

// Cache policy of the weight loads.  Every weight is read once per launch; where every load instruction
// fetches whole 128-byte lines, they are marked non-temporal (nt, bit 1): the lines pass through L2
// without displacing the activations and partial sums (packed decode step 5-8 % faster; row-major
// (28672, 4096) at 16 tokens 44.6 -> 41.0 us).  Packed planes always do; row-major ones if the rows start
// on lines.  Otherwise two pieces share a line, which then has to stay in L2 (K = 4112: 51.8 us with
// the default policy, 58.6 us non-temporal).
constexpr int kStream = 2, kCached = 0;

// 128-byte row pieces per wave, tile and weight array
template <int KIND, int SPW> constexpr int row_pieces() { return kind_is_nested(KIND) ? SPW / 2 : SPW; }

// Packed weights of K-step `S` of the wave's slice.  The whole offset is in the range-checked VGPR part
// of the address (the scalar offset is not range-checked).  va / vb: the lane's columns of the first /
// second 16 bytes lie inside K; otherwise the load is sent out of range and returns zero.
template <int KIND, int POL, int S>
__device__ __forceinline__ void load_w(WItem &r, __amdgpu_buffer_rsrc_t r0, __amdgpu_buffer_rsrc_t r1,
                                       uint32_t voff, bool va, bool vb) {
    typedef WLayout<KIND> L;
    const uint32_t oa = va ? voff : kDead, ob = vb ? voff : kDead;
    r.a = __builtin_amdgcn_raw_buffer_load_b128(r0, oa + S * L::STEP, 0, POL);
    r.b = __builtin_amdgcn_raw_buffer_load_b128(r1, ob + S * L::STEP + L::SECOND, 0, POL);
}

// Row-major weights of one tile as they come: for each piece the rows 0 .. 7 and 8 .. 15 of the tile.
// NestedFP keeps a piece (two K-steps) of the upper plane in the first members of its two steps and
// that of the lower plane in the second ones; the other kinds keep a piece (one K-step) in its step.
// kv[q]: the lane's chunk of piece q lies inside K.
template <int KIND, int SPW, int POL>
__device__ __forceinline__ void load_rows(WItem (&w)[SPW], __amdgpu_buffer_rsrc_t r0, __amdgpu_buffer_rsrc_t r1,
                                          uint32_t lo, uint32_t hi, const bool (&kv)[SPW]) {
    if constexpr (kind_is_nested(KIND)) {
#pragma unroll
        for (int q = 0; q < SPW / 2; ++q) {
            w[2 * q].a = __builtin_amdgcn_raw_buffer_load_b128(r0, (kv[q] ? lo : kDead) + q * 128, 0, POL);
            w[2 * q + 1].a = __builtin_amdgcn_raw_buffer_load_b128(r0, (kv[q] ? hi : kDead) + q * 128, 0, POL);
        }
#pragma unroll
        for (int q = 0; q < SPW / 2; ++q) {
            w[2 * q].b = __builtin_amdgcn_raw_buffer_load_b128(r1, (kv[q] ? lo : kDead) + q * 128, 0, POL);
            w[2 * q + 1].b = __builtin_amdgcn_raw_buffer_load_b128(r1, (kv[q] ? hi : kDead) + q * 128, 0, POL);
        }
    } else {
#pragma unroll
        for (int q = 0; q < SPW; ++q) {
            w[q].a = __builtin_amdgcn_raw_buffer_load_b128(r0, (kv[q] ? lo : kDead) + q * 128, 0, POL);
            w[q].b = __builtin_amdgcn_raw_buffer_load_b128(r0, (kv[q] ? hi : kDead) + q * 128, 0, POL);
        }
    }
}

// Activations of one K-step for 16 tokens (128 bytes per token: 64 FP16 or 128 E4M3 values), in load order;
// zero outside M and K.  They take the same way as row-major weights: in operand order a workgroup's
// 16 x K gather, 16 bytes of 16 rows at a time, cost 0.4-1 us per launch at 16 tokens.
template <int KIND>
__device__ __forceinline__ void load_x(u32x4 &xa, u32x4 &xb, const SmallParams &p, int m, int kb) {
    const u32x4 zero = {0u, 0u, 0u, 0u};
    const bool ok = kb < p.K * (kind_is_fp8(KIND) ? 1 : 2);
    const uint8_t *src = p.X + (int64_t)m * p.x_row_bytes + kb;
    xa = ok && m < p.M ? *reinterpret_cast<const u32x4 *>(src) : zero;
    xb = ok && m + 8 < p.M ? *reinterpret_cast<const u32x4 *>(src + 8 * p.x_row_bytes) : zero;
}

__device__ __forceinline__ half8 as_half8(const u32x4 &v) {
    union { u32x4 u; half8 h; } c;
    c.u = v;
    return c.h;
}

// Turns the raw weight bytes of one step into MFMA operands (merges the planes if nested).
template <int KIND>
__device__ __forceinline__ void prep_w(const WItem &w, u32x4 &w_lo, u32x4 &w_hi) {
    if (kind_is_nested(KIND)) {
        merge16(w.a, w.b, w_lo, w_hi);             // Sec. 4.2, Alg. 1
    } else {
        w_lo = w.a;
        w_hi = w.b;
    }
}

template <int KIND>
__device__ __forceinline__ floatx4 mma_step(const u32x4 &w_lo, const u32x4 &w_hi, const u32x4 &xa,
                                            const u32x4 &xb, floatx4 acc) {
    if (kind_is_fp8(KIND)) {
        intx8 a, b;
        a[0] = w_lo.x; a[1] = w_lo.y; a[2] = w_lo.z; a[3] = w_lo.w;
        a[4] = w_hi.x; a[5] = w_hi.y; a[6] = w_hi.z; a[7] = w_hi.w;
        b[0] = xa.x; b[1] = xa.y; b[2] = xa.z; b[3] = xa.w;
        b[4] = xb.x; b[5] = xb.y; b[6] = xb.z; b[7] = xb.w;
        // E4M3 x E4M3, unit block scales
        return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, acc, 0, 0, 0, 0, 0, 0);
    } else {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_half8(w_lo), as_half8(xa), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_half8(w_hi), as_half8(xb), acc, 0, 0, 0);
        return acc;
    }
}

template <int KIND, int SPW, int POL, int S = 0>
struct FetchTile {
    static __device__ __forceinline__ void run(WItem (&w)[SPW], __amdgpu_buffer_rsrc_t r0,
                                               __amdgpu_buffer_rsrc_t r1, uint32_t voff,
                                               const bool (&va)[SPW], const bool (&vb)[SPW]) {
        if constexpr (KIND == kNestedF16 && S == 0) {
            // packed planes: the tile's blocks of the upper plane first, then those of the lower plane,
            // two runs of consecutive kilobytes instead of an alternation between two distant arrays
            // (about 1 % on the decode step, timed against the plain kernel of the same run as control)
            typedef WLayout<KIND> L;
#pragma unroll
            for (int q = 0; q < SPW; ++q)
                w[q].a = __builtin_amdgcn_raw_buffer_load_b128(r0, (va[q] ? voff : kDead) + q * L::STEP, 0, POL);
#pragma unroll
            for (int q = 0; q < SPW; ++q)
                w[q].b = __builtin_amdgcn_raw_buffer_load_b128(r1, (vb[q] ? voff : kDead) + q * L::STEP + L::SECOND, 0, POL);
        } else {
            load_w<KIND, POL, S>(w[S], r0, r1, voff, va[S], vb[S]);
            FetchTile<KIND, SPW, POL, S + 1>::run(w, r0, r1, voff, va, vb);
        }
    }
};
template <int KIND, int SPW, int POL>
struct FetchTile<KIND, SPW, POL, SPW> {
    static __device__ __forceinline__ void run(WItem (&)[SPW], __amdgpu_buffer_rsrc_t, __amdgpu_buffer_rsrc_t,
                                               uint32_t, const bool (&)[SPW], const bool (&)[SPW]) {}
};

// Activation-stationary streaming kernel.
//   workgroup = up to 16 waves; wave w owns the K-slice [w*SPW*KSTEP, (w+1)*SPW*KSTEP) of
//   grid slice blockIdx.y and keeps the activations of that slice in registers for the whole
//   kernel; the workgroup walks through `tiles_per_wg` 16-row weight tiles, so each wave
//   streams 16 rows x (SPW*KSTEP) contiguous K per tile.  Two tile buffers swap roles
//   (no copies, no branch in the loop body): the loads of tile t+1 are in flight while
//   tile t is merged and multiplied.  Per-tile partial sums go to LDS and are reduced
//   across the waves once, at the end, in fixed wave order.
template <int KIND, int MT, int SPW, bool MULTIPASS, int POL>
__global__ void __launch_bounds__((MT == 4 || SPW == 8) ? 512 : 1024)
small_gemm_kernel(SmallParams p) {
    extern __shared__ float lds[];                    // [tile][wave][MT][64] x float4, then 2 KB per wave
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int waves = blockDim.x >> 6;
    const int g = lane >> 4;
    const int r16 = lane & 15;
    const int slice = blockIdx.y;
    typedef WLayout<KIND> L;
    constexpr int KSTEP = StepK<KIND>::value;
    constexpr int KLANE = 16;                         // first column of lane group g within a step: 16*g
    const int tiles_total = (p.N + 15) >> 4;
    // a workgroup's tiles: a contiguous chunk (stride 1) or interleaved with the other
    // workgroups (stride gridDim.x), so that the chip sweeps the weights front to back
    const int tstride = p.tile_stride;
    const int tile0 = tstride == 1 ? blockIdx.x * p.tiles_per_wg : blockIdx.x;
    const int T = tstride == 1 ? min(p.tiles_per_wg, tiles_total - tile0)
                               : (tiles_total - tile0 + tstride - 1) / tstride;
    floatx4 *slots = reinterpret_cast<floatx4 *>(lds);
    // Which K-slice of the workgroup's this wave takes (see `rotate` in launch_small_gemm; the sums do
    // not depend on it).
    const int ks = !L::PACKED && p.rotate ? (int)((wave + (blockIdx.x >> 3) * 5u) % (unsigned)waves) : wave;
    const __amdgpu_buffer_rsrc_t rs0 = weight_rsrc(p.W0, p.w_bytes);
    const __amdgpu_buffer_rsrc_t rs1 = weight_rsrc(kind_is_nested(KIND) ? p.W1 : p.W0, p.w_bytes);
    const uint32_t tile_bytes = p.tile_bytes;

    // with several K passes this wave's partial tiles live in LDS and start at zero
    // (the spare slot of an odd T included)
    if (MULTIPASS)
        for (int tile = 0; tile < ((T + 1) & ~1); ++tile)
#pragma unroll
            for (int i = 0; i < MT; ++i)
                slots[((tile * waves + ks) * MT + i) * 64 + lane] = floatx4{0.f, 0.f, 0.f, 0.f};

    // Long rows take several passes: in pass q the wave owns K-slice (slice*passes + q)*waves
    // + ks, reloads the activations of that slice and walks the same tiles again, adding
    // to its partial tiles in LDS.
    u32x4 xa[SPW][MT], xb[SPW][MT];
    uint32_t voff = 0;
    bool va[SPW], vb[SPW];                            // packed: this lane's columns of step s lie inside K; row-major: va, of piece s
    const uint32_t own = (uint32_t)(((T + 1) & ~1) * waves * MT * 1024 + wave * 2048);     // behind the slots
    const Regroup<!kind_is_fp8(KIND)> rx(reinterpret_cast<uint8_t *>(lds), own, lane);
    const Regroup<KIND == kPlainF16> rw(reinterpret_cast<uint8_t *>(lds), own, lane);

    auto fetch = [&](WItem (&w)[SPW], int tile) {
        // past the last tile every lane is sent out of range
        const uint32_t base = tile < T ? voff + (uint32_t)(tile0 + tile * tstride) * tile_bytes : kDead;
        if constexpr (L::PACKED) FetchTile<KIND, SPW, POL>::run(w, rs0, rs1, base, va, vb);
        else load_rows<KIND, SPW, POL>(w, rs0, rs1, base, base + 8u * p.w_row_bytes, va);
    };
    auto consume = [&](WItem (&w)[SPW], int tile) {
        floatx4 acc[MT];
        if constexpr (!L::PACKED) {
            if constexpr (kind_is_nested(KIND)) {
#pragma unroll
                for (int s = 0; s < SPW; s += 2) rw.run(w[s].a, w[s + 1].a);
#pragma unroll
                for (int s = 0; s < SPW; s += 2) rw.run(w[s].b, w[s + 1].b);
            } else {
#pragma unroll
                for (int s = 0; s < SPW; ++s) rw.run(w[s].a, w[s].b);
            }
        }
#pragma unroll
        for (int i = 0; i < MT; ++i)
            acc[i] = MULTIPASS ? slots[((tile * waves + ks) * MT + i) * 64 + lane] : floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < SPW; ++s) {
            u32x4 w_lo, w_hi;
            prep_w<KIND>(w[s], w_lo, w_hi);
#pragma unroll
            for (int i = 0; i < MT; ++i) acc[i] = mma_step<KIND>(w_lo, w_hi, xa[s][i], xb[s][i], acc[i]);
        }
#pragma unroll
        for (int i = 0; i < MT; ++i) slots[((tile * waves + ks) * MT + i) * 64 + lane] = acc[i];
    };

    WItem buf0[SPW], buf1[SPW];
    __shared__ uint32_t row_max[kind_quantizes(KIND) ? 16 * 16 : 1];   // per wave and token row
    __shared__ float row_scale[kind_quantizes(KIND) ? 16 : 1];
    const int passes = MULTIPASS ? p.k_passes : 1;
    for (int pass = 0; pass < passes; ++pass) {
        const int k_slice = ((slice * passes + pass) * waves + ks) * (SPW * KSTEP);
        const int k_wave = k_slice + KLANE * g;
        if (L::PACKED) {
            voff = (uint32_t)lane * 16u + (uint32_t)(k_slice >> 6) * (1024u * L::EB);   // block column of the slice
#pragma unroll
            for (int s = 0; s < SPW; ++s) {
                va[s] = k_wave + s * KSTEP < p.K;
                vb[s] = kind_is_fp8(KIND) ? k_wave + s * KSTEP + 64 < p.K : va[s];
            }
        } else {
            const int kb = k_slice * L::EB + (lane & 7) * 16;      // byte column of the lane's chunk of the first piece
            voff = (uint32_t)(lane >> 3) * p.w_row_bytes + (uint32_t)kb;
#pragma unroll
            for (int q = 0; q < SPW; ++q) va[q] = q < row_pieces<KIND, SPW>() && kb + 128 * q < p.K * L::EB;
        }
        if constexpr (kind_quantizes(KIND)) {
            // Activations quantised here (Sec. 2.2 per-token scaling; one token tile, the workgroup covers all of K):
            // every wave loads the FP16 activations of its own slice in load order (lane l: rows l / 8 and 8 + l / 8, 16
            // columns), the row maxima are combined through LDS, each lane converts what it holds -- the
            // quotients and codes of the stand-alone kernel -- and the bytes take the way of loaded ones.
            const int row = lane >> 3;
            constexpr int H = SPW == 2 ? 2 : 1;        // (four K-steps of 16 rows do not fit the registers: M <= 8, see the host)
            const bool two = H == 2 && p.M > 8;
            u32x4 xr[SPW][H][2];
#pragma unroll
            for (int s = 0; s < SPW; ++s) {
                const int k = k_slice + s * KSTEP + 16 * (lane & 7);
                const uint8_t *src = p.X + (int64_t)row * p.x_row_bytes + 2 * (int64_t)k;
                const u32x4 zero = {0u, 0u, 0u, 0u};
                const bool ok = k < p.K && row < p.M, ok2 = k < p.K && row + 8 < p.M;
                xr[s][0][0] = ok ? *reinterpret_cast<const u32x4 *>(src) : zero;
                xr[s][0][1] = ok ? *reinterpret_cast<const u32x4 *>(src + 16) : zero;
                if constexpr (H == 2) {
                    xr[s][1][0] = ok2 ? *reinterpret_cast<const u32x4 *>(src + 8 * p.x_row_bytes) : zero;
                    xr[s][1][1] = ok2 ? *reinterpret_cast<const u32x4 *>(src + 8 * p.x_row_bytes + 16) : zero;
                }
            }
            fetch(buf0, 0);                            // the weights travel during the reduction
            float sc[2], rc[2], rest[2];
            uint32_t largest[2] = {0u, 0u};            // |x| as an integer compare on the magnitude bits
            if (!p.static_scale) {
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    if (h == 1 && !two) break;
#pragma unroll
                    for (int s = 0; s < SPW; ++s)
#pragma unroll
                        for (int q = 0; q < 2; ++q) {
                            const uint32_t w[4] = {xr[s][h][q].x, xr[s][h][q].y, xr[s][h][q].z, xr[s][h][q].w};
#pragma unroll
                            for (int e = 0; e < 4; ++e) largest[h] = max(largest[h], max(w[e] & 0x7fffu, (w[e] >> 16) & 0x7fffu));
                        }
                    largest[h] = max_of_8_lanes(largest[h]);
                    if ((lane & 7) == 0) row_max[wave * 16 + 8 * h + row] = largest[h];
                }
                __syncthreads();
                // (16 waves at most: two words per lane, the maxima of a row's eight lanes)
                const int w0 = min(lane & 7, waves - 1) * 16 + row, w1 = min((lane & 7) + 8, waves - 1) * 16 + row;
                largest[0] = max_of_8_lanes(max(row_max[w0], row_max[w1]));
                if (two) largest[1] = max_of_8_lanes(max(row_max[w0 + 8], row_max[w1 + 8]));
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float amax = half_bits_to_float(largest[h]);
                sc[h] = p.static_scale ? *p.static_scale : (amax == 0.0f ? 1.0f : amax / 448.0f);
                rc[h] = 1.0f / sc[h];                  // correctly rounded; see div_by_scale
                rest[h] = rest_of_reciprocal(sc[h], rc[h]);
                if (wave == 0 && (lane & 7) == 0) row_scale[8 * h + row] = sc[h];
            }
            // (a row with an infinity or a NaN, a scale given by the caller: codes that need clamping)
            const bool plain = p.quant_hw && !p.static_scale && !__any(largest[0] >= 0x7c00u || largest[1] >= 0x7c00u);
#pragma unroll
            for (int s = 0; s < SPW; ++s) {
                auto convert = [&](u32x4 &to, const u32x4 (&x)[2], float sc_, float rc_, float rest_) {
                    if (plain) to = u32x4{quant4_own_scale(x[0].x, x[0].y, rc_, rest_), quant4_own_scale(x[0].z, x[0].w, rc_, rest_),
                                          quant4_own_scale(x[1].x, x[1].y, rc_, rest_), quant4_own_scale(x[1].z, x[1].w, rc_, rest_)};
                    else if (p.quant_hw) to = u32x4{quant4<true>(x[0].x, x[0].y, sc_, rc_), quant4<true>(x[0].z, x[0].w, sc_, rc_),
                                                    quant4<true>(x[1].x, x[1].y, sc_, rc_), quant4<true>(x[1].z, x[1].w, sc_, rc_)};
                    else to = u32x4{quant4<false>(x[0].x, x[0].y, sc_, rc_), quant4<false>(x[0].z, x[0].w, sc_, rc_),
                                    quant4<false>(x[1].x, x[1].y, sc_, rc_), quant4<false>(x[1].z, x[1].w, sc_, rc_)};
                };
                convert(xa[s][0], xr[s][0], sc[0], rc[0], rest[0]);
                xb[s][0] = u32x4{0u, 0u, 0u, 0u};
                if constexpr (H == 2)
                    if (two) convert(xb[s][0], xr[s][1], sc[1], rc[1], rest[1]);
                rx.run(xa[s][0], xb[s][0]);
            }
        } else {
            // (the first weights travel while the activations are regrouped)
#pragma unroll
            for (int s = 0; s < SPW; ++s)
#pragma unroll
                for (int i = 0; i < MT; ++i)
                    load_x<KIND>(xa[s][i], xb[s][i], p, 16 * i + (lane >> 3),
                                 (k_slice + s * KSTEP) * (kind_is_fp8(KIND) ? 1 : 2) + (lane & 7) * 16);
            fetch(buf0, 0);
#pragma unroll
            for (int s = 0; s < SPW; ++s)
#pragma unroll
                for (int i = 0; i < MT; ++i) rx.run(xa[s][i], xb[s][i]);
        }
        // The scheduling barriers keep the compiler from sinking the look-ahead loads below the
        // multiplies (which would turn every wait into a full drain).  For odd T the last
        // half-trip multiplies zeros into a spare slot.
        for (int tile = 0; tile < T; tile += 2) {
            fetch(buf1, tile + 1);
            __builtin_amdgcn_sched_barrier(0);
            consume(buf0, tile);
            __builtin_amdgcn_sched_barrier(0);
            fetch(buf0, tile + 2);
            __builtin_amdgcn_sched_barrier(0);
            consume(buf1, tile + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __syncthreads();

    // ---- fixed-order reduction over the waves of the workgroup -----------------------------
    auto store_y = [&](floatx4 sum, int m, int n) {
        if (kind_is_fp8(KIND)) {
            float sc = (kind_quantizes(KIND) ? row_scale[m] : p.scales[m]) * p.w_scale;
            sum.x = scale_f32(sum.x, sc); sum.y = scale_f32(sum.y, sc); sum.z = scale_f32(sum.z, sc); sum.w = scale_f32(sum.w, sc);
        }
        uint16_t *dst = p.Y + (int64_t)m * p.ldy + n;
        if (p.vec_store && n + 3 < p.N) {
            u32x2 o;
            o.x = float2_to_half2_bits(sum.x, sum.y);
            o.y = float2_to_half2_bits(sum.z, sum.w);
            *reinterpret_cast<u32x2 *>(dst) = o;
        } else {
            float v[4] = {sum.x, sum.y, sum.z, sum.w};
            for (int q = 0; q < 4 && n + q < p.N; ++q) {
                union { _Float16 f; uint16_t u; } cv;
                cv.f = (_Float16)v[q];
                dst[q] = cv.u;
            }
        }
    };
    // Partial sums of a grid-level K split.  Where the last workgroup to arrive finishes the sum
    // (p.counters), they are written through to memory and read back past the caches (cache policy
    // sc0 sc1, system scope): every XCD has an L2 of its own, and the alternative -- a release fence
    // in every workgroup, which writes back the whole L2, and an acquire fence, which invalidates
    // it -- made the kernel four times slower (measured).
    const bool fused = gridDim.y > 1 && p.counters != nullptr;
    constexpr int kThrough = 1 | 16;                  // buffer cache policy: sc0 | sc1
    const int64_t slice_elems = (int64_t)p.M * p.ldp;
    const __amdgpu_buffer_rsrc_t rpart = __builtin_amdgcn_make_buffer_rsrc(
        p.partials, 0, fused ? (uint32_t)(gridDim.y * slice_elems * 4) : 0u, 0x00020000);
    for (int item = wave; item < T * MT; item += waves) {
        const int tile = item / MT, i = item - tile * MT;
        // (eight, four, two reads under way at a time: read one by one, the last seven of 8 or 16 waves cost as many trips to LDS)
        floatx4 sum = slots[((tile * waves) * MT + i) * 64 + lane];
        int w2 = 1;
        auto add = [&](auto count) {
            floatx4 v[decltype(count)::value];
#pragma unroll
            for (int q = 0; q < decltype(count)::value; ++q) v[q] = slots[((tile * waves + w2 + q) * MT + i) * 64 + lane];
#pragma unroll
            for (int q = 0; q < decltype(count)::value; ++q) { sum.x += v[q].x; sum.y += v[q].y; sum.z += v[q].z; sum.w += v[q].w; }
            w2 += decltype(count)::value;
        };
        if (waves - w2 >= 8) add(std::integral_constant<int, 8>{});
        if (waves - w2 >= 4) add(std::integral_constant<int, 4>{});
        if (waves - w2 >= 2) add(std::integral_constant<int, 2>{});
        if (waves - w2 >= 1) add(std::integral_constant<int, 1>{});
        const int m = 16 * i + r16;
        const int n = (tile0 + tile * tstride) * 16 + 4 * g;
        if (m >= p.M || n >= p.N) continue;
        if (gridDim.y > 1) {
            const int64_t e = ((int64_t)slice * p.M + m) * p.ldp + n;
            if (fused)
                __builtin_amdgcn_raw_buffer_store_b128(u32x4{__float_as_uint(sum.x), __float_as_uint(sum.y),
                                                             __float_as_uint(sum.z), __float_as_uint(sum.w)},
                                                       rpart, (uint32_t)(e * 4), 0, kThrough);
            else
                *reinterpret_cast<floatx4 *>(p.partials + e) = sum;
        } else {
            store_y(sum, m, n);
        }
    }
    if (!fused) return;

    // ---- grid-level K split finished by the last workgroup to arrive -------------------------
    // Every workgroup of a tile column waits until its partial sums have reached memory, then takes
    // a ticket; the one that draws the last ticket adds the slices in slice order -- the order of
    // the stand-alone reduction kernel, so the result does not depend on who came last -- and
    // leaves the counter at zero for the next launch.  Nobody waits for anybody.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this lane's write-through stores are done
    __syncthreads();
    uint32_t &ticket = *reinterpret_cast<uint32_t *>(lds);         // (the partial sums in LDS are used up)
    if (threadIdx.x == 0)
        ticket = __hip_atomic_fetch_add(&p.counters[blockIdx.x], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (ticket != gridDim.y - 1) return;
    for (int item = wave; item < T * MT; item += waves) {
        const int tile = item / MT, i = item - tile * MT;
        const int m = 16 * i + r16;
        const int n = (tile0 + tile * tstride) * 16 + 4 * g;
        if (m >= p.M || n >= p.N) continue;
        const uint32_t off = (uint32_t)(((int64_t)m * p.ldp + n) * 4);
        const uint32_t sstep = (uint32_t)(slice_elems * 4);
        // (four slices under way at a time; loads past the last one are sent out of range)
        const int slices = (int)gridDim.y;
        floatx4 sum = {0.f, 0.f, 0.f, 0.f};
        for (int s2 = 0; s2 < slices; s2 += 4) {
            u32x4 v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                v[q] = __builtin_amdgcn_raw_buffer_load_b128(rpart, s2 + q < slices ? off + (uint32_t)(s2 + q) * sstep : 0x80000000u, 0, kThrough);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const floatx4 u = {__uint_as_float(v[q].x), __uint_as_float(v[q].y), __uint_as_float(v[q].z), __uint_as_float(v[q].w)};
                if (s2 + q == 0) sum = u;
                else if (s2 + q < slices) { sum.x += u.x; sum.y += u.y; sum.z += u.z; sum.w += u.w; }
            }
        }
        store_y(sum, m, n);
    }
    if (threadIdx.x == 0) __hip_atomic_store(&p.counters[blockIdx.x], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sums the S split-K partials (rows of ldp floats) in slice order, four columns per lane, applies the
// FP8-mode scale, writes fp16.  VEC: 8-byte stores (N % 4 == 0 and 8-byte aligned output rows).
template <bool VEC>
__global__ void __launch_bounds__(256)
splitk_reduce_kernel(const float *__restrict__ partials, int S, int M, int N, int ldp, const float *scales,
                     float w_scale, uint16_t *__restrict__ Y, int64_t ldy) {
    const int64_t total = (int64_t)M * ldp;
    const int64_t idx = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (idx >= total) return;
    const int m = (int)(idx / ldp), n = (int)(idx - (int64_t)m * ldp);
    floatx4 v = *reinterpret_cast<const floatx4 *>(partials + idx);
    for (int s = 1; s < S; ++s) {
        const floatx4 u = *reinterpret_cast<const floatx4 *>(partials + (int64_t)s * total + idx);
        v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
    }
    if (scales) {
        const float sc = scales[m] * w_scale;
        v.x = scale_f32(v.x, sc); v.y = scale_f32(v.y, sc); v.z = scale_f32(v.z, sc); v.w = scale_f32(v.w, sc);
    }
    uint16_t *dst = Y + (int64_t)m * ldy + n;
    if (VEC) {
        u32x2 o;
        o.x = float2_to_half2_bits(v.x, v.y);
        o.y = float2_to_half2_bits(v.z, v.w);
        *reinterpret_cast<u32x2 *>(dst) = o;
    } else {
        const float x[4] = {v.x, v.y, v.z, v.w};
        for (int q = 0; q < 4 && n + q < N; ++q) {
            union { _Float16 f; uint16_t u; } c;
            c.f = (_Float16)x[q];
            dst[q] = c.u;
        }
    }
}

int launch_splitk_reduce(const float *partials, int S, int64_t M, int64_t N, const float *scales,
                         float w_scale, uint16_t *Y, int64_t ldy, hipStream_t stream) {
    const int64_t ldp = partial_ld(N), total = M * ldp;
    const bool vec = (N & 3) == 0 && (ldy & 3) == 0 && (reinterpret_cast<uintptr_t>(Y) & 7) == 0;
    const unsigned blocks = (unsigned)((total / 4 + 255) / 256);
    if (vec) splitk_reduce_kernel<true><<<blocks, 256, 0, stream>>>(partials, S, (int)M, (int)N, (int)ldp, scales, w_scale, Y, ldy);
    else splitk_reduce_kernel<false><<<blocks, 256, 0, stream>>>(partials, S, (int)M, (int)N, (int)ldp, scales, w_scale, Y, ldy);
    return hip_ok(hipGetLastError());
}

// ---- host-side configuration ---------------------------------------------------------
struct SmallConfig { int mt, spw, waves, split, passes, tiles_per_wg; double cost; };

// Launch shapes of the streaming kernel that were timed faster than what the cost model below chooses, on the
// layer shapes of the models the paper evaluates (Sec. 5.1), for batches of up to 16 tokens.
struct TunedSmall { int cls, N, K, spw, split, tiles; };
static const TunedSmall kTunedSmall[] = {
#include "tuned_small.inc"
    {-1, 0, 0, 0, 0, 0},
};

// What a launch costs, in microseconds.  Fitted by fit_costs.py to 129 000 timings: 72 layer shapes of 0.3 to
// 500 Mi weights x 1, 8, 16, 24, 32 and 64 tokens x both storage orders of the planes and FP16 weights x
// every K split, slice length and tile count; weights cold, replayed graphs.  On those the cheapest candidate
// is 1 % behind the fastest launch on average, 5-6 % at the 95th percentile.  What it says: a K split
// costs about 1 us and 0.7 us per slice (the last workgroup's three trips to memory), more than it gives
// on small layers, where eight slices took 10 us against 4.3 for one ((1560, 1040), 1 token); a CU takes in
// weights at 40 GB/s at most, and at 27 if its workgroups have a single tile each, whose look-ahead then has
// nothing to fetch: (2432, 7104) at 1 token 13.4 us on 152 workgroups of one tile, 10.6 on 228 of two.
struct SmallCost {
    double base;            // launch, first load, reduction over the waves
    double chip_rate, cu_rate;      // bytes per microsecond of the weight stream: whole chip, one CU
    double single;          // a CU's time with one tile per workgroup, against several
    double four;            // a CU's time with four token tiles, against one or two
    double split, slice;    // K split: once, per slice
    double x_rate;          // bytes per microsecond at which a CU fetches activations
    double round;           // workgroups beyond what fits the chip at a time, per round
    double part_rate;       // bytes per microsecond of partial sums
    double pass;            // a further pass over K
};
static const SmallCost kSmallCost[2] = {
    // FP16 mode; plain FP16 too (fitted together), so that the same knobs give both the same launch shape
    {2.90, 8.08e6, 40.4e3, 1.47, 1.25, 0.57, 0.67, 110e3, 2.37, 1.11e6, 1.24},
    {2.99, 8.01e6, 40.6e3, 1.48, 1.34, 0.35, 0.73, 137e3, 1.58, 0.98e6, 1.23},      // E4M3
};

static double price_small(int kind, const SmallConfig &c, int64_t M, int64_t N, int64_t K) {
    const bool fp8 = kind_is_fp8(kind);
    const SmallCost &k = kSmallCost[fp8 ? 1 : 0];
    const double wb = fp8 ? 1.0 : 2.0;                            // bytes per weight, and per activation
    const int64_t tiles = (N + 15) / 16;
    const int64_t wgs = ((tiles + c.tiles_per_wg - 1) / c.tiles_per_wg) * c.split;
    const int64_t lds = (int64_t)((c.tiles_per_wg + 1) & ~1) * c.waves * c.mt * 1024 + c.waves * 2048;
    const int waves_cu = c.mt == 1 ? (c.spw == 2 ? 28 : (c.spw == 4 ? 16 : 8)) : (c.mt == 2 ? 20 : 16);   // by registers
    const int64_t slots = std::max<int64_t>(1, std::min<int64_t>(160 * 1024 / lds, waves_cu / c.waves));
    const double k_wg = (double)c.waves * c.passes * c.spw * (fp8 ? 128 : 64);      // columns of a workgroup
    const double wg_cu = (double)((wgs + 255) / 256);             // workgroups of the busiest CU
    const double chip = (double)N * (double)K * wb / k.chip_rate;
    const double cu = wg_cu * c.tiles_per_wg * 16.0 * std::min(k_wg, (double)K) * wb / k.cu_rate *
                      (c.tiles_per_wg == 1 ? k.single : 1.0) * (c.mt == 4 ? k.four : 1.0);
    const double a = chip * chip, b = cu * cu;
    double t = k.base + std::sqrt(std::sqrt(a * a + b * b));
    t += wg_cu * (double)std::min<int64_t>(M, 16 * c.mt) * k_wg * wb / k.x_rate;
    t += k.round * (double)((wgs + 256 * slots - 1) / (256 * slots) - 1) + k.pass * (c.passes - 1);
    if (c.split > 1) t += k.split + k.slice * c.split + (double)c.split * (double)M * (double)N * 4.0 / k.part_rate;
    return t;
}

static SmallConfig compute_small(int kind, int64_t M, int64_t N, int64_t K) {
    const Tuning &t = tuning();
    const int mt = M <= 16 ? 1 : (M <= 32 ? 2 : 4);
    // knobs first; with none set, the table of timed shapes; otherwise the cheapest candidate
    int64_t k_spw = t.small_spw, k_split = t.small_split, k_tiles = t.small_tiles;
    if (k_spw <= 0 && k_split <= 0 && k_tiles <= 0 && t.tuned_table != 0 && mt == 1) {
        for (const TunedSmall &e : kTunedSmall)
            if (e.cls == kind_class(kind) && e.N == N && e.K == K) {
                k_spw = e.spw;  k_split = e.split;  k_tiles = e.tiles;
                break;
            }
    }
    const bool fp8 = kind_is_fp8(kind);
    const int kstep = fp8 ? 128 : 64;
    const int steps = (int)((K + kstep - 1) / kstep);
    // K-steps per wave: 2 or 4; 2 with several token tiles (their activations need the registers); 8 where
    // it is asked for and exists (row-major weights of a long K: 512 bytes or more of each row)
    const bool can_long = (kind == kPlainF16 || kind == kNestedF16Row) && mt == 1 && (K + 63) / 64 >= 64;
    int spws[2] = {2, 4}, n_spw = 2;
    if (mt > 1) n_spw = 1;
    else if (k_spw == 2 || k_spw == 4 || (k_spw == 8 && can_long)) { spws[0] = (int)k_spw;  n_spw = 1; }
    else if (k_spw == 8) { spws[0] = 4;  n_spw = 1; }
    SmallConfig best;
    best.cost = 1e30;
    for (int q = 0; q < n_spw; ++q) {
        SmallConfig c;
        c.mt = mt;
        c.spw = spws[q];
        const int max_waves = (mt == 4 || c.spw == 8) ? 8 : 16;   // (these need up to 256 VGPRs per wave)
        const int slices = (steps + c.spw - 1) / c.spw;           // wave-sized K slices
        const int rounds = (slices + max_waves - 1) / max_waves;
        for (int split : {1, 2, 3, 4, 6, 8}) {
            if (k_split > 0) split = (int)std::min<int64_t>(k_split, slices);
            // a split's scratch has to leave room in the fixed scratch of nestedfp_gemm_static, which takes
            // every problem that fits it unsplit
            else if (split > 1 && (split > slices || (double)split * (double)M * (double)N * 4.0 +
                                                     (fp8 ? (double)M * (double)K : 0.0) > 30.0 * 1024 * 1024)) break;
            // what the waves of all grid slices do not cover at once is walked in passes
            c.split = split;
            c.passes = (rounds + split - 1) / split;
            c.waves = (slices + split * c.passes - 1) / (split * c.passes);
            // a workgroup keeps a kilobyte of partial sums per tile, token tile and wave in LDS (an even
            // number of tiles, 128 KB at most)
            int per_max = (128 / (c.waves * mt)) & ~1;
            per_max = std::max(1, std::min(per_max, 16));
            for (int per = 1; per <= per_max; ++per) {
                c.tiles_per_wg = k_tiles > 0 ? (int)std::min<int64_t>(k_tiles, per_max) : per;
                c.cost = price_small(kind, c, M, N, K);
                if (c.cost < best.cost) best = c;
                if (k_tiles > 0) break;
            }
            if (k_split > 0) break;
        }
    }
    return best;
}

static SmallConfig choose_small(int kind, int64_t M, int64_t N, int64_t K) {
    static thread_local PlanCache<SmallConfig> cache;
    // (row-major planes can take 8 K-steps where packed ones cannot)
    return cache.get(kind == kNestedF16Row ? 3 : kind_class(kind), M, N, K, [&] { return compute_small(kind, M, N, K); });
}

double small_gemm_cost(int kind, int64_t M, int64_t N, int64_t K) { return choose_small(kind, M, N, K).cost; }

bool small_gemm_supports(int kind, int64_t M, int64_t N, int64_t K, int64_t ldw) {
    // the weight array must be addressable with 31-bit byte offsets (bit 31 marks a load as dead),
    // a few tiles of slack included
    (void)M;
    return weight_array_bytes(kind, N + 48, K, ldw) < ((int64_t)1 << 31);
}

size_t small_gemm_partial_bytes(int kind, int64_t M, int64_t N, int64_t K) {
    SmallConfig c = choose_small(kind, M, N, K);
    return c.split > 1 ? (size_t)c.split * (size_t)M * (size_t)partial_ld(N) * sizeof(float) : 0;
}

// dynamic LDS of a launch: a kilobyte per tile, token tile and wave (an even number of tiles), 2 KB per wave to regroup in
static size_t small_lds(const SmallConfig &c) {
    return (size_t)((c.tiles_per_wg + 1) & ~1) * c.waves * c.mt * 1024 + (size_t)c.waves * 2048;
}
constexpr int kQuantLds = 158 * 1024;                            // (the row maxima and scales are static)

template <int KIND, int MT, int SPW, int POL = kStream>
static void launch_small_t(const SmallParams &p, const SmallConfig &c, dim3 grid, hipStream_t stream) {
    if constexpr (!kind_is_packed(KIND) && POL == kStream) {      // rows that do not start on lines (see kStream)
        if ((p.w_row_bytes & 127) != 0 || (reinterpret_cast<uintptr_t>(p.W0) & 127) != 0 ||
            (reinterpret_cast<uintptr_t>(p.W1) & 127) != 0) {
            launch_small_t<KIND, MT, SPW, kCached>(p, c, grid, stream);
            return;
        }
    }
    const size_t lds = small_lds(c);
    constexpr bool passes = !kind_quantizes(KIND);               // (quantising kinds have one pass)
    auto kern1 = small_gemm_kernel<KIND, MT, SPW, false, POL>;
    auto kernp = small_gemm_kernel<KIND, MT, SPW, passes, POL>;
    static std::atomic<bool> attr_set{false};                    // once per instantiation
    if (!attr_set.load(std::memory_order_acquire)) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern1),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, passes ? 160 * 1024 : kQuantLds);
        if (passes) (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kernp),
                                              hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        attr_set.store(true, std::memory_order_release);
    }
    if (c.passes > 1) kernp<<<grid, c.waves * 64, lds, stream>>>(p);
    else kern1<<<grid, c.waves * 64, lds, stream>>>(p);
}

// Whether the streaming kernel quantises the activations itself: one token tile, all of K in the workgroup.  What it saves
// is a launch (1.3 us in a graph, 3 us of host time outside one); what it costs is that every workgroup waits for
// its M x K activations, their row maxima and 3 VALU instructions per value before it multiplies, while two weight
// tiles are on their way.  Up to 8 tokens (half the lanes' rows) that pays where a workgroup has further tiles or the
// rows are short (us with the launch of its own / fused): (1024, 1024) 5.2 / 4.0, (12288, 3072) 10.9 / 9.8, (8192, 5120) 11.6 / 11.0,
// (8192, 8192) 15.7 / 14.9; with one tile (4096, 4096) takes 8.5 / 8.5 and (3072, 7168) 10.5 / 11.3.  With 16 rows to convert it pays
// on short rows, 16 tokens on (1024, 1280) 5.8 / 5.5, and up to 3584 columns from three tiles on: (12288, 2048) 9.6 / 9.0,
// (32768, 2048) 15.2 / 14.7, (16384, 3584) 14.2 / 13.7 at 9 tokens and level at 16, (6144, 2560) with two 8.0 / 8.4, (4096, 4096) 8.7 / 10.5.
bool small_gemm_fuses_quant(int64_t M, int64_t N, int64_t K) {
    const int64_t knob = tuning().small_fuse_quant;
    if (knob == 0) return false;
    const SmallConfig c = choose_small(kE4M3, M, N, K);
    if (c.mt != 1 || c.split != 1 || c.passes != 1 || (c.spw != 2 && M > 8) || small_lds(c) > (size_t)kQuantLds) return false;
    return knob > 0 || (M <= 8 ? (c.tiles_per_wg > 1 || K <= 3072) : (K <= 1280 || (K <= 3584 && c.tiles_per_wg > 2)));
}

template <int KIND>
static void launch_small_k(const SmallParams &p, const SmallConfig &c, dim3 grid, hipStream_t stream) {
    if constexpr (KIND == kPlainF16 || KIND == kNestedF16Row) {
        if (c.mt == 1 && c.spw == 8) { launch_small_t<KIND, 1, 8>(p, c, grid, stream);  return; }
    }
    if constexpr (kind_quantizes(KIND)) {                        // (one token tile)
        if (c.spw == 4) launch_small_t<KIND, 1, 4>(p, c, grid, stream);
        else launch_small_t<KIND, 1, 2>(p, c, grid, stream);
    } else {
        switch (c.mt * 10 + c.spw) {
            case 14: launch_small_t<KIND, 1, 4>(p, c, grid, stream); break;
            case 12: launch_small_t<KIND, 1, 2>(p, c, grid, stream); break;
            case 22: launch_small_t<KIND, 2, 2>(p, c, grid, stream); break;
            default: launch_small_t<KIND, 4, 2>(p, c, grid, stream); break;
        }
    }
}

int launch_small_gemm(int kind, const GemmArgs &a, hipStream_t stream) {
    SmallConfig c = choose_small(kind, a.M, a.N, a.K);
    SmallParams p;
    p.X = static_cast<const uint8_t *>(a.X);
    p.x_row_bytes = (kind == kE4M3 || kind == kE4M3Row) ? a.ldx : 2 * a.ldx;
    p.scales = a.scales;
    p.static_scale = a.static_scale;
    p.quant_hw = tuning().quant_hw != 0 ? 1 : 0;
    p.w_scale = a.w_scale;
    p.W0 = static_cast<const uint8_t *>(a.W0);
    p.W1 = static_cast<const uint8_t *>(a.W1);
    if (kind_is_packed(kind)) {
        // 16 rows of a tile take 16 * Kp contiguous elements (Kp = K rounded up to 64)
        p.w_row_bytes = 0;
        p.tile_bytes = (uint32_t)(((a.K + 63) / 64) * 1024 * kind_elem_bytes(kind));
    } else {
        p.w_row_bytes = (uint32_t)(kind == kPlainF16 ? 2 * a.ldw : a.K);
        p.tile_bytes = 16u * p.w_row_bytes;
    }
    p.w_bytes = (uint32_t)weight_array_bytes(kind, a.N, a.K, a.ldw);
    p.M = (int)a.M;  p.N = (int)a.N;  p.K = (int)a.K;
    p.Y = a.Y;  p.ldy = a.ldy;
    p.partials = a.partials;
    p.ldp = (int)partial_ld(a.N);
    p.tiles_per_wg = c.tiles_per_wg;
    const int64_t tiles = (a.N + 15) / 16;
    const unsigned grid_x = (unsigned)((tiles + c.tiles_per_wg - 1) / c.tiles_per_wg);
    // the last workgroup of a tile column sums the K slices itself where there is a counter for it
    const bool fused_reduce = c.split > 1 && a.counters != nullptr && grid_x <= (unsigned)kMaxCounters &&
                              (int64_t)c.split * a.M * partial_ld(a.N) * 4 < ((int64_t)1 << 32) && tuning().fused_reduce != 0;
    p.counters = fused_reduce ? a.counters : nullptr;
    p.k_passes = c.passes;
    p.tile_stride = (tuning().small_interleave != 0 && c.tiles_per_wg > 1) ? (int)grid_x : 1;
    // Rows that are a multiple of 4 KB long put the 16 rows of a slice on the same memory channels, and as
    // the workgroups start together, wave by wave, the whole chip asks for one group of channels after
    // the other; with the slices rotated from workgroup to workgroup of an XCD it does not (16 tokens,
    // FP16 mode: (28672, 4096) 44.2 -> 39.5 us, (57344, 8192) 174 -> 154 us).  Other row lengths lose up to
    // 3 % by it, and plain FP16 weights, whose slices are a kilobyte long, gain only from rows of 16 KB on
    // ((57344, 8192) 172 -> 150 us, (28672, 4096) 37.2 -> 38.4 us).
    const uint32_t channels = kind == kPlainF16 ? 16384u : 4096u;
    p.rotate = !kind_is_packed(kind) && p.w_row_bytes % channels == 0 ? 1 : 0;
    p.vec_store = ((a.N & 3) == 0 && (a.ldy & 3) == 0 && (reinterpret_cast<uintptr_t>(a.Y) & 7) == 0) ? 1 : 0;
    if (c.split > 1 && (a.partials == nullptr ||
                        a.partial_bytes < (size_t)c.split * a.M * partial_ld(a.N) * sizeof(float)))
        return kErrWorkspace;
    dim3 grid(grid_x, (unsigned)c.split);
    if (kind_quantizes(kind) && !(c.mt == 1 && c.split == 1 && c.passes == 1)) return kErrArg;   // caller checks first
    switch (kind) {
        case kPlainF16: launch_small_k<kPlainF16>(p, c, grid, stream); break;
        case kPlainF16Packed: launch_small_k<kPlainF16Packed>(p, c, grid, stream); break;
        case kNestedF16: launch_small_k<kNestedF16>(p, c, grid, stream); break;
        case kNestedF16Row: launch_small_k<kNestedF16Row>(p, c, grid, stream); break;
        case kE4M3Quant: launch_small_k<kE4M3Quant>(p, c, grid, stream); break;
        case kE4M3QuantRow: launch_small_k<kE4M3QuantRow>(p, c, grid, stream); break;
        case kE4M3Row: launch_small_k<kE4M3Row>(p, c, grid, stream); break;
        case kE4M3: launch_small_k<kE4M3>(p, c, grid, stream); break;
        default: return kErrArg;
    }
    if (hipGetLastError() != hipSuccess) return kErrHip;
    if (c.split > 1 && !fused_reduce)
        return launch_splitk_reduce(a.partials, c.split, a.M, a.N, kind_is_fp8(kind) ? a.scales : nullptr,
                                    a.w_scale, a.Y, a.ldy, stream);
    return kOk;
}

}  // namespace nfp
