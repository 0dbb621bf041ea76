// Per-token activation quantisation to E4M3 for FP8 mode (Sec. 2.2 "E4M3 Format",
// Sec. 5.1 "Methodology").  One workgroup per token row: pass 1 finds the row's largest
// magnitude, pass 2 (the row is still in cache) divides and converts.  HBM-bound:
// 2 bytes read + 1 byte written per activation.
#include "nfp_device.h"
#include "nfp_host.h"

namespace nfp {

constexpr int kQuantThreads = 256;

// Decode-sized batches wait for one chain: launch, load, maximum, conversion, store.  Maxima go by DPP, those of the waves are
// read in one LDS access, and rows of finite activations take the short conversion.  Replayed in a graph, before and now: 16 tokens of
// 4096 columns 2.63 -> 2.33 us, of 14336 3.90 -> 2.99; 777 tokens 4.2 -> 3.8 and 10.4 -> 8.0; 8192 tokens 19.5 -> 18.6 and 73 -> 63.
struct RowScale { float s, y, rest;  bool plain; };
template <bool HW>
__device__ __forceinline__ RowScale scale_of(const float *static_scale, uint32_t amax_bits) {
    RowScale r;
    const float amax = half_bits_to_float(amax_bits);
    r.s = static_scale ? *static_scale : (amax == 0.0f ? 1.0f : amax / 448.0f);
    r.y = 1.0f / r.s;                                // correctly rounded; see div_by_scale
    r.rest = rest_of_reciprocal(r.s, r.y);
    r.plain = HW && !static_scale && amax_bits < 0x7c00u;     // (an infinity or a NaN, a scale given by the caller: codes that need clamping)
    return r;
}
// the maximum of a workgroup of `waves` waves, red: a word for each
__device__ __forceinline__ uint32_t max_of_workgroup(uint32_t v, uint32_t *red, int waves) {
    v = max_of_wave(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)max_of_16_lanes(red[min((int)(threadIdx.x & 15), waves - 1)]));
}
template <bool HW>
__device__ __forceinline__ u32x2 quant8(const u32x4 &v, const RowScale &r) {
    if (r.plain) return u32x2{quant4_own_scale(v.x, v.y, r.y, r.rest), quant4_own_scale(v.z, v.w, r.y, r.rest)};
    return u32x2{quant4<HW>(v.x, v.y, r.s, r.y), quant4<HW>(v.z, v.w, r.s, r.y)};
}

template <bool HW>
__global__ void __launch_bounds__(kQuantThreads)
quantize_act_kernel(const uint16_t *__restrict__ X, int64_t K, int64_t ldx,
                    const float *__restrict__ static_scale, uint8_t *__restrict__ Xq,
                    float *__restrict__ scales, int64_t ldq) {
    const int64_t m = blockIdx.x;
    const u32x4 *row = reinterpret_cast<const u32x4 *>(X + m * ldx);
    const int chunks = (int)(K / 8);                 // 8 halves per 16-byte chunk
    __shared__ uint32_t red[kQuantThreads / 64];
    uint32_t amax_bits = 0;
    if (!static_scale) {
        // |x| as an integer compare on the magnitude bits: monotone for finite halves
        for (int c = threadIdx.x; c < chunks; c += kQuantThreads) {
            u32x4 v = row[c];
            uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t lo = w[i] & 0x7fffu, hi = (w[i] >> 16) & 0x7fffu;
                amax_bits = max(amax_bits, max(lo, hi));
            }
        }
        amax_bits = max_of_workgroup(amax_bits, red, kQuantThreads / 64);
    }
    const RowScale r = scale_of<HW>(static_scale, amax_bits);
    if (threadIdx.x == 0) scales[m] = r.s;
    u32x2 *out = reinterpret_cast<u32x2 *>(Xq + m * ldq);
    for (int c = threadIdx.x; c < chunks; c += kQuantThreads) out[c] = quant8<HW>(row[c], r);
}

// Single-pass variant for rows that fit in registers (K <= 32768): every lane keeps its
// 16-byte chunks between the maximum and the conversion, so the row is read once and the
// kernel is one load latency shorter -- what matters for decode-sized batches, where this
// kernel is pure latency, and for long rows, whose second read no longer comes from the cache.
template <int CPT, bool HW>
__global__ void __launch_bounds__(1024)
quantize_act_onepass_kernel(const uint16_t *__restrict__ X, int64_t K, int64_t ldx,
                            const float *__restrict__ static_scale, uint8_t *__restrict__ Xq,
                            float *__restrict__ scales, int64_t ldq) {
    const int64_t m = blockIdx.x;
    const u32x4 *row = reinterpret_cast<const u32x4 *>(X + m * ldx);
    const int chunks = (int)(K / 8);
    __shared__ uint32_t red[16];
    u32x4 v[CPT];
    uint32_t amax_bits = 0;
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        int c = threadIdx.x + i * blockDim.x;
        v[i] = c < chunks ? row[c] : u32x4{0u, 0u, 0u, 0u};
        uint32_t w[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
        for (int q = 0; q < 4; ++q) amax_bits = max(amax_bits, max(w[q] & 0x7fffu, (w[q] >> 16) & 0x7fffu));
    }
    if (!static_scale) amax_bits = max_of_workgroup(amax_bits, red, blockDim.x >> 6);
    const RowScale r = scale_of<HW>(static_scale, amax_bits);
    if (threadIdx.x == 0) scales[m] = r.s;
    u32x2 *out = reinterpret_cast<u32x2 *>(Xq + m * ldq);
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        int c = threadIdx.x + i * blockDim.x;
        if (c < chunks) out[c] = quant8<HW>(v[i], r);
    }
}

template <int CPT>
static void launch_onepass(bool hw, int threads, const uint16_t *X, int64_t M, int64_t K, int64_t ldx,
                           const float *static_scale, uint8_t *Xq, int64_t ldq, float *scales, hipStream_t stream) {
    dim3 grid((unsigned)M);
    if (hw)
        quantize_act_onepass_kernel<CPT, true><<<grid, threads, 0, stream>>>(X, K, ldx, static_scale, Xq, scales, ldq);
    else
        quantize_act_onepass_kernel<CPT, false><<<grid, threads, 0, stream>>>(X, K, ldx, static_scale, Xq, scales, ldq);
}

int launch_quantize_act(const uint16_t *X, int64_t M, int64_t K, int64_t ldx,
                        const float *static_scale, uint8_t *Xq, int64_t ldq, float *scales, hipStream_t stream) {
    bool hw = tuning().quant_hw != 0;
    const int64_t chunks = K / 8;
    const int64_t onepass = tuning().quant_onepass;
    // one pass for decode-sized batches (latency; at 300 to 500 tokens still 3.8 against 4.1 us for K = 4096, 5.0 against
    // 5.5 for 7168, and 4.8 against 5.2 at 1000 tokens for 4096, where 7168 takes 8.0 against 7.4) and for long
    // rows at any batch (measured at 8192 tokens: 5.1-5.4 TB/s against 3.9 for K = 14336 / 28672, equal at
    // K = 8192, 4 % behind at 4096)
    const bool few = M <= 512 || (M <= 1024 && chunks <= 512);
    if (chunks <= 4096 && (onepass > 0 || (onepass < 0 && (few || chunks >= 1024)))) {
        // as many lanes as the row has chunks (up to 1024, 4 chunks each)
        int cpt = chunks <= 1024 ? 1 : (chunks <= 2048 ? 2 : 4);
        int threads = (int)(((chunks + cpt - 1) / cpt + 63) / 64 * 64);
        if (cpt == 1) launch_onepass<1>(hw, threads, X, M, K, ldx, static_scale, Xq, ldq, scales, stream);
        else if (cpt == 2) launch_onepass<2>(hw, threads, X, M, K, ldx, static_scale, Xq, ldq, scales, stream);
        else launch_onepass<4>(hw, threads, X, M, K, ldx, static_scale, Xq, ldq, scales, stream);
        return hip_ok(hipGetLastError());
    }
    dim3 grid((unsigned)M);
    if (hw)
        quantize_act_kernel<true><<<grid, kQuantThreads, 0, stream>>>(X, K, ldx, static_scale, Xq, scales, ldq);
    else
        quantize_act_kernel<false><<<grid, kQuantThreads, 0, stream>>>(X, K, ldx, static_scale, Xq, scales, ldq);
    return hip_ok(hipGetLastError());
}

}  // namespace nfp
