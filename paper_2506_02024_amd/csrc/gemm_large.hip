// LDS-tiled MFMA GEMMs for prefill-sized batches: Y = X * W^T, compute-bound.
//
// Four kernels.  large_gemm_kernel multiplies plain FP16 weights or E4M3 weights (FP8 mode: the
// upper plane as it is, row-major or in packed blocks): TM tokens x TN weight rows x 128 bytes of K
// per row (64 halves or 128 E4M3 bytes) per stage, two or more LDS stages, 8 waves.  nested_bypass_kernel is FP16 mode: Sec. 4.2
// puts the FP16 reconstruction between the shared-memory-to-register copy and the tensor-core
// instruction of every warp and hides it with a third pipeline stage; here every weight belongs
// to exactly one wave, which loads its 16 bytes of each plane per lane (from row-major planes or
// from packed blocks) into registers, merges them there (Alg. 1) and feeds them to the MFMA -- the
// weights never pass through LDS; the same kernel without the merge multiplies FP16 weights stored
// in packed blocks, the like-for-like baseline of Sec. 5.2.  nested_rows_kernel is FP16 mode on row-major planes, which
// come by whole lines through a part of the LDS that belongs to the wave.  e4m3_bypass_kernel
// is the same register path for E4M3 weights, used for batches of 49 .. 64 tokens, where the
// weight stream is the bound.
//
// In all of them, weight rows are the MFMA "A" operand and tokens the "B" operand, so a lane holds 4
// consecutive output columns of one token.  Tokens and plain / E4M3 weights reach LDS by
// direct-to-LDS buffer loads; FP16 rows are 128 bytes with the 16-byte chunk index XOR-swizzled
// with the row so that the MFMA fragment reads are free of bank conflicts, packed E4M3 blocks
// are copied as they are.
#include <type_traits>

#include "nfp_device.h"
#include "nfp_host.h"

namespace nfp {

struct LargeParams {
    const uint8_t *X;       // fp16 X (bytes) or E4M3 Xq
    int64_t x_row_bytes;    // 256 rows of it stay below 2^31 (checked on the host): bit 31 of a tile-local offset marks a dead load
    const float *scales;
    float w_scale;
    const uint8_t *W0;
    const uint8_t *W1;
    int64_t w_row_bytes;    // bytes per row of W0 for row-major weights (plain: 2*ldw, planes / E4M3: K); same limit
    int M, N, K;
    int k_bytes;            // bytes per row along K for 8-chunk operands (2K or K)
    int kblocks;            // 64-column blocks per row tile of a packed plane: ceil(K / 64)
    uint16_t *Y;
    int64_t ldy;
    float *partials;        // rows of ldp floats (see partial_ld)
    int ldp;
    int tiles_m, tiles_n;
    int ktiles_total, ktiles_per_split;
    int rows_anywhere;      // output rows need not start on 16 bytes (N or ldy no multiple of 8, or Y not 16-byte aligned)
    int xcd_map;            // group the token tiles of a weight tile on one XCD (see tile_of_block)
    int xcd_group;          // token tiles per group of an XCD's part; 0: another order
};

// Which tile a workgroup takes.  The hardware deals consecutive workgroups to the 8 XCDs in turn,
// and every XCD has an L2 of its own.  In launch order "token tile fastest" the token tiles of one weight tile land on
// different XCDs, and each of those fetches the weights from memory again.
// Up to seven token tiles: workgroup b of XCD b % 8 takes token tile (b / 8) % tiles_m of weight tile
// 8 * ((b / 8) / tiles_m) + b % 8, so that all token tiles of a weight tile follow each other on one XCD.  The last
// tiles_n % 8 weight tiles keep the launch order.
// From eight on (p.xcd_group): every XCD takes an eighth of the tiles, in an order that runs through groups of up to
// six token tiles, all weight tiles of a group before the next: the 32 tiles that an XCD has under way are about six by
// six, 12 operand tiles to fetch.  In launch order they are that only where tiles_m is a multiple of 8; else every XCD
// has all token tiles under way, and with 9 or more of them it fetches up to three times as much.  Timed in turn on 26 000 launches
// (150 layers, 80 to 8192 tokens, weights cold), time against the launch order, FP16 mode and FP8 mode: 9 to 15 token
// tiles 0.96 and 0.92, 16 0.98 and 0.96, 17 to 23 0.97 and 0.95, 24 1.0, 25 to 31 0.90 and 0.89, 32 0.99 and 0.96, 33 and
// more 0.93 and 0.90; 8 against the order of fewer 0.99.  Groups of 8 or 16 are 1-4 % behind groups of 6; fewer than eight
// token tiles as one group: level.
__device__ __forceinline__ void tile_of_block(const LargeParams &p, int b, int &tm, int &tn) {
    if (p.xcd_group) {
        const int total = p.tiles_m * p.tiles_n, x = b & 7;
        const int v = x * (total >> 3) + min(x, total & 7) + (b >> 3);       // the first total % 8 XCDs have one tile more
        const int g = v / (p.xcd_group * p.tiles_n), u = v - g * (p.xcd_group * p.tiles_n);
        const int rows = min(p.xcd_group, p.tiles_m - g * p.xcd_group);
        tn = u / rows;
        tm = g * p.xcd_group + u - tn * rows;
        return;
    }
    const int grouped = 8 * p.tiles_m * (p.tiles_n >> 3);
    if (p.xcd_map && b < grouped) {
        const int j = b >> 3;
        tm = j % p.tiles_m;
        tn = (j / p.tiles_m) * 8 + (b & 7);
    } else if (p.xcd_map) {
        const int r = b - grouped;
        tm = r % p.tiles_m;
        tn = (p.tiles_n & ~7) + r / p.tiles_m;
    } else {
        tm = b % p.tiles_m;
        tn = b / p.tiles_m;
    }
}

// LDS tiles are rows of 128 bytes; the 16-byte chunk index is XOR-ed with (row >> 1) & 7.
// gfx950 serves ds_read_b128 at 256 B/clk only if 16 consecutive lanes hit 64 distinct
// 4-byte banks: rows r, r+1 then share a swizzle and fill one 256-byte bank line, and the
// pairs of 16 consecutive rows take the 8 different swizzles.  The 128-bit writes of the
// global->LDS copy (8 lanes per row) are conflict-free under the same map.
__device__ __forceinline__ int swz(int row, int chunk) { return row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4); }

// FP16 tiles: which 16-byte chunk of a 128-byte global row the physical chunk slot p of an LDS row
// holds (before the XOR swizzle).  The sum over k does not care about the order of k as long as
// both operands agree.  The register-path NestedFP kernel gets its weights 16 consecutive columns
// per lane (lane group g = l / 16 holds columns 16 g .. 16 g + 15 of a packed block), so substep
// s of a K-tile multiplies halves 16 g + 8 s .. + 7, i.e. chunk 2 g + s of the row; all FP16 kernels
// use that order, so that they add up alike and FP16 mode equals the plain FP16 GEMM bit for bit.
// In LDS the four lane groups must read ADJACENT chunks (a stride of two chunks between the
// groups halves the LDS read rate: bank conflicts), so chunk 2 g + s is stored in slot 4 s + g.
__device__ __forceinline__ int fp16_chunk_of_slot(int p) { return ((p & 3) << 1) | (p >> 2); }

__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const uint8_t *base, int64_t row0, int rows,
                                                            int64_t row_bytes, int k_bytes) {
    // raw buffer over the rows of one tile; anything past the last valid byte reads as zero
    uint32_t bytes = rows > 0 ? (uint32_t)((rows - 1) * row_bytes + k_bytes) : 0u;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(base + row0 * row_bytes), 0, bytes, 0x00020000);
}

// The K loops load a few K-tiles ahead.  Past the end of a workgroup's K-slice those loads are sent out of
// range like the ones past K: nobody uses them, and a slice of 16 K-tiles would otherwise fetch 2 to 4
// of the next slice's as well.  Returns the slice's end in bytes of a row of tokens (128 per K-tile).
__device__ __forceinline__ uint32_t slice_end(const LargeParams &p, int kt_end) {
    return (uint32_t)min((int64_t)p.k_bytes, (int64_t)kt_end * 128);
}

// raw buffer over the 16-row tiles of a packed plane (blocks of block_bytes) that hold rows row0 .. row0+rows-1
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const uint8_t *base, int64_t row0, int rows, int kblocks,
                                                             int block_bytes) {
    const int64_t tile_bytes = (int64_t)kblocks * block_bytes;
    uint32_t bytes = rows > 0 ? (uint32_t)(((rows + 15) >> 4) * tile_bytes) : 0u;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(base + (row0 >> 4) * tile_bytes), 0, bytes, 0x00020000);
}

// ---- writing a workgroup's result tile ------------------------------------------------------------
// MB: rows of an MFMA block (16 or 32).  Accumulator layout: lane l holds token l % MB of a block
// and, for v = 0 .. MB*MB/256 - 1, the four consecutive weight rows
// (MB == 32 ? 8 v + 4 (l / 32) : 4 (l / 16)) .. +3.
template <int KIND, int TM, int TN, int WAVES_M, int WAVES_N, int MB_ = (kind_is_fp8(KIND) ? 32 : 16)>
struct TileStore {
    static constexpr int WAVES = WAVES_M * WAVES_N;
    static constexpr int WTM = TM / WAVES_M, WTN = TN / WAVES_N;
    static constexpr int MB = MB_;
    static constexpr int FMB = (WTM + MB - 1) / MB, FNB = WTN / MB;      // (WTM: on average, see LargeKernel::UNEVEN)
    typedef typename std::conditional<MB == 32, floatx16, floatx4>::type AccT;

    // Result tile through LDS: the MFMA layout leaves a lane with 4 consecutive outputs of one
    // token, so direct stores are 8-byte pieces scattered over 16 or 32 rows per instruction.  Written
    // to LDS as FP16 first (16-byte chunks XOR-swizzled with the row), the tile goes out as
    // whole rows, 16 bytes per lane, every store instruction covering complete 128-byte lines.
    // The caller guarantees that no wave still reads the operand stages.
    static constexpr int OCH = TN * 2 / 16;            // 16-byte chunks per output row
    static constexpr int NV = MB == 32 ? 4 : 1;
    static __device__ __forceinline__ float scaled(float x, float s) { return kind_is_fp8(KIND) ? scale_f32(x, s) : x; }
    static __device__ __forceinline__ int acc_col(int lane, int v) { return MB == 32 ? 8 * v + 4 * (lane >> 5) : 4 * (lane >> 4); }

    // row0: the wave's first token row within the tile, F: its token blocks
    template <int F>
    static __device__ __forceinline__ void to_lds(const LargeParams &p, AccT (&acc)[FNB][FMB], int m0, int row0, int wn, int lane,
                                                  uint8_t *lds) {
        const int r = lane % MB;
#pragma unroll
        for (int j = 0; j < F; ++j) {
            const int row = row0 + MB * j + r;
            float s = 1.0f;
            if (kind_is_fp8(KIND)) {
                const int m = m0 + row;
                s = (m < p.M ? p.scales[m] : 0.f) * p.w_scale;
            }
#pragma unroll
            for (int i = 0; i < FNB; ++i)
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const int col = wn * WTN + MB * i + acc_col(lane, v);
                    const int chunk = col >> 3;
                    u32x2 o;
                    o.x = float2_to_half2_bits(scaled(acc[i][j][4 * v], s), scaled(acc[i][j][4 * v + 1], s));
                    o.y = float2_to_half2_bits(scaled(acc[i][j][4 * v + 2], s), scaled(acc[i][j][4 * v + 3], s));
                    *reinterpret_cast<u32x2 *>(lds + row * (TN * 2) + ((chunk ^ (row & (OCH - 1))) << 4) + 8 * ((col >> 2) & 1)) = o;
                }
        }
    }
    static __device__ __forceinline__ void epilogue_lds(const LargeParams &p, AccT (&acc)[FNB][FMB], int m0, int n0,
                                                        int row0, int wn, int lane, int wave, uint8_t *lds) {
        to_lds<FMB>(p, acc, m0, row0, wn, lane, lds);
        __syncthreads();
        store_rows(p, m0, n0, lane, wave, lds);
    }
    static __device__ __forceinline__ void store_rows(const LargeParams &p, int m0, int n0, int lane, int wave, const uint8_t *lds) {
        constexpr int RPI = 64 / OCH;                  // rows per store instruction
        constexpr int ROWS = TM / WAVES;               // rows per wave
        const int chunk = lane % OCH;
        if (p.rows_anywhere) {
            store_rows_shifted(p, m0, n0, lane, wave, lds);
            return;
        }
        const int n = n0 + chunk * 8;
#pragma unroll
        for (int it = 0; it < ROWS / RPI; ++it) {
            const int row = wave * ROWS + it * RPI + lane / OCH;
            const u32x4 v = *reinterpret_cast<const u32x4 *>(lds + row * (TN * 2) + ((chunk ^ (row & (OCH - 1))) << 4));
            const int m = m0 + row;
            if (m < p.M && n < p.N) *reinterpret_cast<u32x4 *>(p.Y + (int64_t)m * p.ldy + n) = v;
        }
    }

    // Output rows that start anywhere (N or ldy no multiple of 8): a row's first 16-byte boundary lies `skip` columns
    // into the tile, and the 16 bytes that a lane stores are put together from two chunks of the LDS.  The columns
    // before the first boundary and behind the last go out two bytes at a time, those of 8 rows per instruction.
    // Straight from the MFMA layout, in two-byte pieces, a lane needs four stores for what is one here: FP8 mode
    // (7955, 1280) at 1768 tokens 62.7 us so, 32.0 through LDS; (28689, 4096) at 777 tokens 154 and 101, at 200 tokens 51.7 and
    // 42.2; FP16 mode (12479, 2304) at 2048 tokens 155 and 125, at 100 tokens 24.7 and 23.1.  N = 28676, whose rows took
    // 8-byte pieces: level at 2048 tokens (432 us packed).
    static __device__ __forceinline__ void store_rows_shifted(const LargeParams &p, int m0, int n0, int lane, int wave, const uint8_t *lds) {
        constexpr int RPI = 64 / OCH, ROWS = TM / WAVES;
        const int chunk = lane % OCH;
        const int n_end = min(p.N, n0 + TN);
#pragma unroll
        for (int it = 0; it < ROWS / RPI; ++it) {
            const int row = wave * ROWS + it * RPI + lane / OCH, m = m0 + row;
            uint16_t *const dst = p.Y + (int64_t)m * p.ldy + n0;
            const int skip = (int)(0u - (uint32_t)(reinterpret_cast<uintptr_t>(dst) >> 1)) & 7;
            const uint8_t *const src = lds + row * (TN * 2);
            const u32x4 a = *reinterpret_cast<const u32x4 *>(src + ((chunk ^ (row & (OCH - 1))) << 4));
            const u32x4 b = *reinterpret_cast<const u32x4 *>(src + (((chunk + 1) & (OCH - 1)) ^ (row & (OCH - 1))) * 16);
            // eight dwords, moved down by four bytes times skip / 2, then by two more if skip is odd
            const bool four = (skip & 4) != 0, two = (skip & 2) != 0;
            const uint32_t t0 = four ? a.z : a.x, t1 = four ? a.w : a.y, t2 = four ? b.x : a.z, t3 = four ? b.y : a.w,
                           t4 = four ? b.z : b.x, t5 = four ? b.w : b.y;
            const uint32_t u0 = two ? t1 : t0, u1 = two ? t2 : t1, u2 = two ? t3 : t2, u3 = two ? t4 : t3, u4 = two ? t5 : t4;
            const uint32_t half = (uint32_t)(skip & 1) * 16u;
            const u32x4 v = {__builtin_amdgcn_alignbit(u1, u0, half), __builtin_amdgcn_alignbit(u2, u1, half),
                             __builtin_amdgcn_alignbit(u3, u2, half), __builtin_amdgcn_alignbit(u4, u3, half)};
            const int c = skip + 8 * chunk, n = n0 + c;
            if (m < p.M && c + 8 <= TN) {
                if (n + 8 <= n_end) *reinterpret_cast<u32x4 *>(dst + c) = v;
                else if (n < n_end) store_some(dst + c, v, n_end - n);
            }
        }
        // (skip = 0: the row is whole 16-byte pieces)
#pragma unroll
        for (int it = 0; it < (ROWS + 7) / 8; ++it) {
            const int r = it * 8 + (lane >> 3), row = wave * ROWS + r, m = m0 + row;
            uint16_t *const dst = p.Y + (int64_t)m * p.ldy + n0;
            const int skip = (int)(0u - (uint32_t)(reinterpret_cast<uintptr_t>(dst) >> 1)) & 7;
            const int c = (lane & 7) < skip ? lane & 7 : TN - 8 + (lane & 7);
            if (r < ROWS && m < p.M && skip != 0 && n0 + c < n_end)
                dst[c] = *reinterpret_cast<const uint16_t *>(lds + row * (TN * 2) + (((c >> 3) ^ (row & (OCH - 1))) << 4) + 2 * (c & 7));
        }
    }
    // the first `count` < 8 of eight halves
    static __device__ __forceinline__ void store_some(uint16_t *dst, const u32x4 &v, int count) {
#pragma unroll
        for (int q = 0; q < 7; ++q)
            if (q < count) dst[q] = (uint16_t)(v[q >> 1] >> (16 * (q & 1)));
    }

    // A slice's sums of a K split, straight from the MFMA layout: 16 bytes per lane.  (Outputs have the one way through LDS only: a
    // second one straight from here, though never taken, cost a quarter of the tiled kernels' code and the row-major 256 x 256 kernel
    // of FP16 mode four more spilled registers; 2048 tokens of a Llama-3 8B layer 844 us with it, 838 without.)
    template <int F = FMB>
    static __device__ __forceinline__ void store_partials(const LargeParams &p, AccT (&acc)[FNB][FMB], int m0, int n0,
                                                          int row0, int wn, int lane, int split) {
        const int r = lane % MB;
#pragma unroll
        for (int j = 0; j < F; ++j) {
            const int m = m0 + row0 + MB * j + r;
            if (m >= p.M) continue;
#pragma unroll
            for (int i = 0; i < FNB; ++i)
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const int n = n0 + wn * WTN + MB * i + acc_col(lane, v);
                    if (n < p.N)
                        *reinterpret_cast<floatx4 *>(p.partials + ((int64_t)split * p.M + m) * p.ldp + n) =
                            floatx4{acc[i][j][4 * v], acc[i][j][4 * v + 1], acc[i][j][4 * v + 2], acc[i][j][4 * v + 3]};
                }
        }
    }
};

// NST: LDS stages.  Two are enough where two workgroups share a CU; a launch with at most one workgroup per CU takes
// three or four on tiles below 256 x 256, so that loads run NST - 1 K-tiles ahead.
// NSTW: stages of the weights.  On 256 x 256 tiles two stages of both and a third one of the weights alone take the
// 160 KB: tokens come from L2, within a K-tile, weights from memory, in two.  With two of both, a K-tile took at least the
// latency of a weight load: FP8 mode, (28672, 4096) at 777 tokens 107 -> 98 us, at 8192 tokens 787 -> 754, (4096, 14336) at
// 300 tokens unsplit 148 -> 107; plain FP16 (4096, 14336) at 2048 tokens unsplit 283 -> 238.
template <int KIND, int TM, int TN, int WAVES_M, int WAVES_N, int NST = 2, int NSTW = NST>
struct LargeKernel {
    static_assert(KIND == kPlainF16 || KIND == kE4M3 || KIND == kE4M3Row, "NestedFP16 has a kernel of its own");
    static constexpr bool FP8 = kind_is_fp8(KIND);
    static constexpr bool PACKED_W = KIND == kE4M3;    // weight stage = packed 1 KB blocks as they are
    static constexpr int WAVES = WAVES_M * WAVES_N;
    static_assert(WAVES == 8, "two waves per SIMD: one loading (older), one not");
    static constexpr int THREADS = 64 * WAVES;
    static constexpr int WTM = TM / WAVES_M, WTN = TN / WAVES_N;
    static constexpr int XSTAGE = TM * 128, WSTAGE = TN * 128;       // bytes per LDS stage
    static constexpr int XBASE = NSTW * WSTAGE;        // the token stages follow the weights'
    static constexpr int LDS_BYTES = XBASE + NST * XSTAGE;
    static_assert(NST >= 2 && (NSTW == NST || NSTW == NST + 1) && LDS_BYTES <= 160 * 1024, "LDS stages");
    typedef TileStore<KIND, TM, TN, WAVES_M, WAVES_N> Store;
    static_assert(TM * TN * 2 <= LDS_BYTES, "output tile must fit into the operand stages");

    // ---- MFMA tiling ------------------------------------------------------------------------
    // FP16 kinds: v_mfma_f32_16x16x32_f16.  Under the chip's power limit (which, not the issue
    // rate, bounds a full-chip FP16 GEMM on random operands) it sustains about 15 % more flops
    // than 32x32x16: it moves half as many accumulator registers per flop.  E4M3:
    // v_mfma_scale_f32_32x32x64_f8f6f4 (the 16x16x128 shape would need more fragment registers
    // than a wave with a 128x64 tile has).  A wave's tile is FNB x FMB blocks of MB weight rows x
    // MB tokens; a K-tile (128 bytes per row) is two substeps of 64 bytes per row; a fragment is
    // NCH 16-byte chunks per lane: lane l supplies row l % MB and bytes 16 * NCH * (l / MB) .. of
    // the substep's 64.
    static constexpr int MB = FP8 ? 32 : 16;
    static constexpr int SUBS = 2;
    static constexpr int NCH = FP8 ? 2 : 1;
    // UNEVEN: tiles of 160 and 224 tokens, an odd number of 32-token blocks for two waves: the older four waves,
    // which issue the loads as well, take one block less than the younger four (two waves of a SIMD are one of each).
    static constexpr bool UNEVEN = WTM % MB != 0;
    static_assert(!UNEVEN || (WAVES_M == 2 && WAVES_N == 4), "one wave of each kind per SIMD");
    static constexpr int FMB = (WTM + MB - 1) / MB, FNB = WTN / MB;
    template <bool OLDER> static constexpr int blocks() { return UNEVEN && OLDER ? FMB - 1 : FMB; }
    typedef typename std::conditional<MB == 32, floatx16, floatx4>::type AccT;
    // Slot plan of a substep.  The MFMAs run token block by token block (the FNB weight
    // fragments stay, the token fragments stream).  The first NPRE fragments of a substep (all
    // weight fragments, up to two token fragments) are fetched in the tail of the substep before
    // it, the other token fragments early in the substep itself, about two token blocks ahead of
    // their use.  The one barrier of a K-tile sits in its second substep behind the last read of
    // the current stage (slot QB): from there on the stage is free for K-tile kt+2; the loads of
    // kt+2 and the first reads of kt+1 follow it.
    template <int F> struct Plan {                                   // F: token blocks of the wave
        static constexpr int MF = F * FNB;                           // MFMAs per substep
        static constexpr int NB0 = F < 2 ? F : 2;
        static constexpr int NPRE = FNB + NB0;
        static constexpr int NREST = F - NB0;
        static constexpr int RSTR = (3 * FNB) / 4 > 0 ? (3 * FNB) / 4 : 1;        // slots between the early token reads
        static constexpr int QB = NREST > 0 ? (NREST - 1) * RSTR + (MB == 32 ? 2 : 3) : 0;   // slot that starts with the barrier
        static constexpr int RPT = (NPRE + (MF - QB) - 1) / (MF - QB);            // look-ahead reads per tail slot
        static constexpr int TSLOTS = (NPRE + RPT - 1) / RPT;                     // tail slots that read
        static constexpr int TSTR = (MF - QB) / TSLOTS;                           // slots between them
        static constexpr int TAIL0 = MF - TSLOTS * TSTR;
        static_assert(QB < MF && TAIL0 >= QB && TSTR >= 1, "slot plan");
    };

    struct Frags { intx4 a[FNB][NCH]; intx4 b[FMB][NCH]; };

    // the chunk slot of an LDS row that lane group g reads in substep s (see fp16_chunk_of_slot)
    static __device__ __forceinline__ int k_chunk(int s, int g, int q) { return 4 * s + NCH * g + q; }

    // LDS address of chunk q of a weight fragment: row, substep s, lane group g = l / MB.
    // Row-major weights: rows of 128 bytes, XOR-swizzled.  Packed E4M3: the stage holds the 1 KB blocks
    // as they are in memory, [row tile][2 blocks]; a substep is one block, and 16 lanes with
    // consecutive rows read 256 consecutive bytes.
    static __device__ __forceinline__ int w_addr(int row, int s, int g, int q) {
        if (PACKED_W) return (((row >> 4) * 2 + s) << 10) + (((row & 15) + 16 * (NCH * g + q)) << 4);
        return swz(row, k_chunk(s, g, q));
    }

    // fragment R of substep s in the order of first use: weight blocks 0..FNB-1, token blocks 0..FMB-1
    template <int R>
    static __device__ __forceinline__ void read_frag(Frags &f, const uint8_t *wstage, const uint8_t *xstage, int row0, int wn, int lane, int s) {
        const int r = lane % MB, g = lane / MB;
#pragma unroll
        for (int q = 0; q < NCH; ++q) {
            if constexpr (R < FNB)
                f.a[R][q] = *reinterpret_cast<const intx4 *>(wstage + w_addr(wn * WTN + MB * R + r, s, g, q));
            else
                f.b[R - FNB][q] = *reinterpret_cast<const intx4 *>(
                    xstage + swz(row0 + MB * (R - FNB) + r, k_chunk(s, g, q)));
        }
    }

    template <int R, int END>
    static __device__ __forceinline__ void read_frags(Frags &f, const uint8_t *wstage, const uint8_t *xstage, int row0, int wn, int lane, int s) {
        if constexpr (R < END) {
            read_frag<R>(f, wstage, xstage, row0, wn, lane, s);
            read_frags<R + 1, END>(f, wstage, xstage, row0, wn, lane, s);
        }
    }

    // weight rows are the "A" operand, tokens the "B" operand: a lane gets one token of the block
    // and groups of four consecutive weight rows
    template <int Q>
    static __device__ __forceinline__ void mfma_one(const Frags &f, AccT (&acc)[FNB][FMB]) {
        constexpr int j = Q / FNB, i = Q % FNB;
        if constexpr (FP8) {
            intx8 a = {f.a[i][0].x, f.a[i][0].y, f.a[i][0].z, f.a[i][0].w, f.a[i][NCH - 1].x, f.a[i][NCH - 1].y, f.a[i][NCH - 1].z, f.a[i][NCH - 1].w};
            intx8 b = {f.b[j][0].x, f.b[j][0].y, f.b[j][0].z, f.b[j][0].w, f.b[j][NCH - 1].x, f.b[j][NCH - 1].y, f.b[j][NCH - 1].z, f.b[j][NCH - 1].w};
            acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc[i][j], 0, 0, 0, 0, 0, 0);
        } else {
            union { intx4 v; half8 h; } a, b;
            a.v = f.a[i][0];
            b.v = f.b[j][0];
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a.h, b.h, acc[i][j], 0, 0, 0);
        }
    }

    // ---- direct-to-LDS loads (buffer_load ... lds) -------------------------------------------
    // One wave instruction fills 1 KB of LDS = 8 tile rows in lane order (lane l -> row l/8,
    // physical chunk l%8), so the XOR swizzle is applied on the global side: lane l fetches
    // the logical chunk (l%8) ^ ((row>>1)&7) of its row.  No VGPR staging, no ds_write.
    // With two waves per SIMD the older one wins every arbitration and reaches the barrier long
    // before the younger one.  The loads are therefore issued by the older four waves only:
    // a load instruction blocks the issue of whatever is behind it while the address queue is
    // full, and those waves have the time to spare.
    static constexpr int DW = 4;                       // waves that issue direct-to-LDS loads
    static constexpr int XG = TM / 8 / DW;             // 8-row groups per loading wave, token tile
    static constexpr int WG8 = TN / 8 / DW;            // 8-row groups per loading wave, weight tile
    static constexpr int DMAS = XG + WG8;              // loads per loading wave per K-tile

    struct DmaOffsets {
        uint32_t x[XG], w[WG8];
        uint32_t kpos;                                 // this lane's K byte position in a K-tile
        int wbit;                                      // E4M3: which of a K-tile's two block columns this wave loads
    };

    static __device__ __forceinline__ void make_dma_offsets(DmaOffsets &o, const LargeParams &p, int wave, int lane) {
        const int pc = lane & 7;
        const int slot = pc ^ ((((wave & 1) << 2) + (lane >> 4)) & 7);  // (row >> 1) & 7 for row = gid*8 + lane/8
        const int c = FP8 ? slot : fp16_chunk_of_slot(slot);
        o.kpos = 16u * c;
#pragma unroll
        for (int i = 0; i < XG; ++i) o.x[i] = (uint32_t)((i * DW + wave) * 8 + (lane >> 3)) * (uint32_t)p.x_row_bytes + 16u * c;
#pragma unroll
        for (int i = 0; i < WG8; ++i) {
            if (PACKED_W) {
                // packed upper plane: load i of wave w is block b = i*DW + w of the stage, i.e. block
                // column (2*kt + b%2) of row tile b/2; lane l fetches chunk l
                const int b = i * DW + wave;
                o.w[i] = (uint32_t)((b >> 1) * p.kblocks + (b & 1)) * 1024u + 16u * lane;
            } else {
                o.w[i] = (uint32_t)((i * DW + wave) * 8 + (lane >> 3)) * (uint32_t)p.w_row_bytes + 16u * c;
            }
        }
        o.wbit = wave & 1;
    }

    typedef __attribute__((address_space(3))) uint8_t lds_byte;

    // the i-th of a wave's XG + WG8 direct-to-LDS loads of one K-tile (token rows first, of K-tile kt into stage xst, weights of
    // ktw into wst);
    // i is a constant at every call site
    static __device__ __forceinline__ void dma_one(int i, const DmaOffsets &o, uint32_t x_lim, uint32_t w_lim,
                                                   __amdgpu_buffer_rsrc_t rx, __amdgpu_buffer_rsrc_t rw,
                                                   lds_byte *lds3, int xst, int wst, int wave, int kt, int ktw) {
        if (i < XG) {
            const uint32_t kb = (uint32_t)kt * 128u;
            const uint32_t kill = (kb + o.kpos < x_lim) ? 0u : 0x80000000u;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (__attribute__((address_space(3))) void *)(lds3 + XBASE + xst * XSTAGE + (i * DW + wave) * 1024),
                                                     16, (o.x[i] + kb) | kill, 0, 0, 0);
        } else {
            const int j = i - XG;
            const uint32_t kb = (uint32_t)ktw * 128u;
            lds_byte *stage = lds3 + wst * WSTAGE;
            if (PACKED_W) {
                // w_lim = block columns of the plane; past them the load is sent out of range
                const uint32_t kill = ((uint32_t)(2 * ktw + o.wbit) < w_lim) ? 0u : 0x80000000u;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (__attribute__((address_space(3))) void *)(stage + (j * DW + wave) * 1024),
                                                         16, (o.w[j] + (uint32_t)ktw * 2048u) | kill, 0, 0, 0);
            } else {
                const uint32_t kill = (kb + o.kpos < w_lim) ? 0u : 0x80000000u;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (__attribute__((address_space(3))) void *)(stage + (j * DW + wave) * 1024),
                                                         16, (o.w[j] + kb) | kill, 0, 0, 0);
            }
        }
    }

    // ---- the K loop as an explicit instruction schedule ---------------------------------------
    // Every MFMA is followed by the few other instructions assigned to its slot and a scheduling
    // fence, so the order below is the order in the binary.  OLDER: one of the DW waves that
    // issue the direct-to-LDS loads; the loop exists once per role so that it has no branches
    // inside.  PAR: which of the two fragment sets the substep multiplies.
    struct Ctx {
        AccT (&acc)[FNB][FMB];
        Frags (&fr)[2];
        const DmaOffsets &dof;
        __amdgpu_buffer_rsrc_t rx, rw;
        uint8_t *lds;
        lds_byte *lds3;
        uint32_t x_lim, w_lim;
        int wave, lane, row0, wn;                       // row0: the wave's first token row
        int kt, cur, nxt, wcur, wnxt;                   // K-tile, its token and weight stages, the next K-tile's
    };

    template <bool OLDER, int S, int PAR, int Q>
    static __device__ __forceinline__ void slot(Ctx &c) {
        typedef Plan<blocks<OLDER>()> P;
        constexpr int MF = P::MF, QB = P::QB, RSTR = P::RSTR, NREST = P::NREST, NPRE = P::NPRE;
        constexpr int DPS = (DMAS + (MF - QB) - 1) / (MF - QB);        // loads per slot behind the barrier
        constexpr bool last = (S == SUBS - 1);
        if constexpr (last && Q == QB) {
            // every read of the current stage has been issued; once all waves are here and their
            // loads of the next K-tile have landed (those of the NST - 2 K-tiles after it, and a further stage of
            // weights, may stay in flight), the stage is free and the next one complete
            if constexpr (OLDER) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NST - 2) * DMAS + (NSTW > NST ? WG8 : 0)) : "memory");
            else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if constexpr (NSTW == 2) {
                __syncthreads();
            } else {
                // a bare barrier: the fence of __syncthreads() would drain the loads in flight.  What
                // it would order is ordered by the waits above: the next stage's loads have landed,
                // and every LDS read of the stage that is refilled next has returned.
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        mfma_one<Q>(c.fr[PAR], c.acc);
        if constexpr (Q % RSTR == 0 && Q / RSTR < NREST)
            read_frag<FNB + P::NB0 + Q / RSTR>(c.fr[PAR], c.lds + c.wcur * WSTAGE, c.lds + XBASE + c.cur * XSTAGE, c.row0, c.wn, c.lane, S);
        if constexpr (Q >= P::TAIL0 && (Q - P::TAIL0) % P::TSTR == 0 && (Q - P::TAIL0) / P::TSTR < P::TSLOTS) {
            constexpr int r0 = (Q - P::TAIL0) / P::TSTR * P::RPT;
            read_frags<r0, (r0 + P::RPT < NPRE ? r0 + P::RPT : NPRE)>(c.fr[PAR ^ 1], c.lds + (last ? c.wnxt : c.wcur) * WSTAGE,
                                                                c.lds + XBASE + (last ? c.nxt : c.cur) * XSTAGE, c.row0, c.wn,
                                                                c.lane, last ? 0 : S + 1);
        }
        if constexpr (last && OLDER && Q >= QB) {
#pragma unroll
            for (int d = (Q - QB) * DPS; d < (Q - QB + 1) * DPS && d < DMAS; ++d)
                dma_one(d, c.dof, c.x_lim, c.w_lim, c.rx, c.rw, c.lds3, c.cur, c.wcur, c.wave, c.kt + NST, c.kt + NSTW);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (Q + 1 < MF) slot<OLDER, S, PAR, Q + 1>(c);
    }

    template <bool OLDER>
    static __device__ __forceinline__ void k_loop(Ctx &c, int kt_begin, int kt_end) {
        int cur = 0, wcur = 0;
        for (int kt = kt_begin; kt < kt_end; ++kt) {
            c.kt = kt;
            c.cur = cur;
            cur = cur + 1 == NST ? 0 : cur + 1;
            c.nxt = cur;
            c.wcur = NSTW == NST ? c.cur : wcur;
            wcur = wcur + 1 == NSTW ? 0 : wcur + 1;
            c.wnxt = NSTW == NST ? c.nxt : wcur;
            __builtin_amdgcn_sched_barrier(0);
            slot<OLDER, 0, 0, 0>(c);
            slot<OLDER, 1, 1, 0>(c);
        }
    }

    static __device__ __forceinline__ void run(const LargeParams &p, uint8_t *lds, lds_byte *lds3) {
        const int lane = threadIdx.x & 63;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int wm = UNEVEN ? wave / WAVES_N : wave % WAVES_M, wn = UNEVEN ? wave % WAVES_N : wave / WAVES_M;
        const int row0 = UNEVEN ? wm * blocks<true>() * MB : wm * WTM;
        int tm, tn;
        tile_of_block(p, blockIdx.x, tm, tn);
        const int m0 = tm * TM, n0 = tn * TN;
        const int split = blockIdx.y;
        const int kt_begin = split * p.ktiles_per_split;
        const int kt_end = min(kt_begin + p.ktiles_per_split, p.ktiles_total);

        const __amdgpu_buffer_rsrc_t rx = tile_rsrc(p.X, m0, min(TM, p.M - m0), p.x_row_bytes, p.k_bytes);
        const __amdgpu_buffer_rsrc_t rw = PACKED_W
            ? plane_rsrc(p.W0, n0, min(TN, p.N - n0), p.kblocks, 1024)
            : tile_rsrc(p.W0, n0, min(TN, p.N - n0), p.w_row_bytes, p.k_bytes);
        DmaOffsets dof;
        make_dma_offsets(dof, p, wave, lane);
        // (no load ahead of the K loop reaches into the next slice of a split: see slice_end)
        const uint32_t x_lim = slice_end(p, kt_end);
        const uint32_t w_lim = PACKED_W ? (uint32_t)min(p.kblocks, 2 * kt_end) : x_lim;

        // Tokens and weights go straight from global memory into LDS.
        if (wave < DW) {
#pragma unroll
            for (int st = 0; st < NSTW; ++st)
#pragma unroll
                for (int i = st < NST ? 0 : XG; i < DMAS; ++i)
                    dma_one(i, dof, x_lim, w_lim, rx, rw, lds3, st, st, wave, kt_begin + st, kt_begin + st);
        }
        // the loads of K-tile kt_begin (a wave that issued none passes straight through)
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 1) * DMAS + (NSTW - NST) * WG8) : "memory");
        if constexpr (NSTW == 2) {
            __syncthreads();
        } else {
            asm volatile("" ::: "memory");                     // (a bare barrier, as in the loop)
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }

        AccT acc[FNB][FMB];
#pragma unroll
        for (int i = 0; i < FNB; ++i)
#pragma unroll
            for (int j = 0; j < FMB; ++j)
#pragma unroll
                for (int q = 0; q < (MB == 32 ? 16 : 4); ++q) acc[i][j][q] = 0.f;
        Frags fr[2];
        Ctx c{acc, fr, dof, rx, rw, lds, lds3, x_lim, w_lim, wave, lane, row0, wn, kt_begin, 0, 0, 0, 0};
        static_assert(Plan<blocks<true>()>::NPRE == Plan<blocks<false>()>::NPRE, "the first fragments are read before the roles part");
        read_frags<0, Plan<FMB>::NPRE>(fr[0], lds, lds + XBASE, row0, wn, lane, 0);
        if (wave < DW) k_loop<true>(c, kt_begin, kt_end);
        else k_loop<false>(c, kt_begin, kt_end);
        // the loads of the K-tiles past the end are still in flight: they must have landed
        // before the LDS is reused for the output tile or handed back
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (gridDim.y == 1) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the look-ahead fragment reads
            __syncthreads();
            if (UNEVEN && wave < DW) Store::template to_lds<blocks<true>()>(p, acc, m0, row0, wn, lane, lds);
            else Store::template to_lds<FMB>(p, acc, m0, row0, wn, lane, lds);
            __syncthreads();
            Store::store_rows(p, m0, n0, lane, wave, lds);
        } else if (UNEVEN && wave < DW) {
            Store::template store_partials<blocks<true>()>(p, acc, m0, n0, row0, wn, lane, split);
        } else {
            Store::template store_partials<FMB>(p, acc, m0, n0, row0, wn, lane, split);
        }
    }
};

template <int KIND, int TM, int TN, int WAVES_M, int WAVES_N, int NST, int NSTW>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N)
large_gemm_kernel(LargeParams p) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
    typedef LargeKernel<KIND, TM, TN, WAVES_M, WAVES_N, NST, NSTW> Kern;
    Kern::run(p, lds_raw, (typename Kern::lds_byte *)lds_raw);
}

// ---- NestedFP16 with the weights kept out of LDS ------------------------------------------------
// Eight waves side by side along the weight rows: a wave owns TN/8 weight rows and all TM tokens
// of the tile, so every weight is needed by exactly one wave.  The wave loads 16 bytes of each
// plane per lane straight into registers (lane l: row l % 16, columns 16 * (l / 16) .. +15 of a
// 64-column block -- one contiguous kilobyte per instruction from packed planes; row-major ones by
// 128-byte pieces of 8 rows, regrouped through LDS, see PAIR), merges them there (Sec. 4.2, Alg. 1) and feeds the result to the MFMA
// as it is (WK = kPlainF16Packed: FP16 weights in packed blocks, no merge): the sum over k
// does not care about the order of k, so substep s of a K-tile takes columns 16 g + 8 s .. + 7
// from lane group g, and the token fragments are read from LDS in the same order (chunk
// 2 g + s of the 128-byte row, see fp16_chunk_of_slot).  No ds_write, no weight tile in LDS; LDS holds four stages of
// the token tile only (loads run three K-tiles ahead), and the one barrier per K-tile sits
// at its end and waits for no LDS read.
// DEEP: a ring of eight token stages with the token loads six and the plane loads four K-tiles ahead
// (tiles of at most 128 tokens, launches that do not fill the chip: there a K-tile's MFMAs are
// short against the latency of a load) instead of four stages and three / two K-tiles.
template <int TM, int TN, int WK, bool DEEP = false, bool NT = false, bool PAIRS = false>
struct BypassKernel {
    static_assert(WK == kNestedF16 || WK == kNestedF16Row || WK == kPlainF16Packed, "weights that go through registers");
    static constexpr bool MERGE = kind_is_nested(WK);
    static constexpr bool ROWMAJOR = WK == kNestedF16Row;
    // NT: the launch has one token tile, so every weight is read once; packed blocks (whole lines per
    // instruction) are then marked non-temporal, as in the streaming kernel.  The 64-token tiles of such a launch always
    // are (and some of several token tiles: see streams_tiles64); the 128-token
    // tiles on the large layers (timed: 6-10 % faster from about 100 Mi weights on at
    // M = 96 and 128, a few per cent slower on the small ones).
    static constexpr int POLICY = NT ? 2 : 0;
    // PAIR: row-major planes are fetched for two K-tiles at a time, 128 bytes of 8 rows per instruction, and
    // regrouped through 2 KB of LDS per wave one K-tile before the first of the two is merged.  Fetched
    // for one K-tile, 64 bytes of 16 rows per instruction, every line is requested twice: (28672, 5120) at 48
    // tokens took 77 us against 56 from packed planes, and takes 60 so.  It costs 16 registers for the second
    // pair and as many for the longer loop, which a wave with 32 weight rows does not have (and which leave
    // room for one workgroup per CU instead of two; capped to 128 registers the kernel is 3 % slower).
    static constexpr bool PAIR = PAIRS;
    static_assert(!PAIR || (ROWMAJOR && TN == 128), "pairs of K-tiles: row-major planes, 16 weight rows per wave");
    static constexpr int BLOCK_BYTES = 1024 * kind_elem_bytes(WK);   // packed kinds: one 16 x 64 block
    typedef TileStore<kNestedF16, TM, TN, 1, 8> Store;
    static constexpr int DW = 4;                               // waves that issue the token loads
    static constexpr int WTN = TN / 8;
    static constexpr int FMB = TM / 16, FNB = WTN / 16;
    static constexpr int MF = FMB * FNB;                       // MFMAs per substep
    // (a ring of eight stages with the token loads six and the plane loads three K-tiles ahead was
    // no faster for the 64-token tiles)
    static constexpr int NST = DEEP ? 8 : 4;                   // LDS stages of the token tile
    static constexpr int XA = DEEP ? 6 : 3;                    // token loads run this many K-tiles ahead
    static constexpr int NRAW = DEEP || PAIR ? 4 : 2;          // register sets of plane blocks, one K-tile each: loaded this many K-tiles ahead
    static_assert(XA >= 3 && XA < NST && (NRAW <= XA || PAIR) && NRAW >= 2, "the stage being filled is neither the one in use nor the next");
    static_assert(NST * TM * 128 <= 160 * 1024, "LDS stages");
    static constexpr int STAGE = TM * 128;
    static constexpr int RING_BYTES = NST * STAGE > TM * TN * 2 ? NST * STAGE : TM * TN * 2;
    static constexpr int LDS_BYTES = RING_BYTES + (PAIR ? 8 * 2048 : 0);     // (behind the ring: 2 KB per wave to regroup in)
    static_assert(LDS_BYTES <= 160 * 1024, "LDS");
    static constexpr int RGS = FMB / 2;                        // PAIR: slots between the 2 FNB regroupings of a pair
    static constexpr int XG = TM / 8 / DW;                     // loads per loading wave per K-tile
    static constexpr int LEAD = 2;                             // token fragments are read this many blocks ahead
    static constexpr int NMQ = 2 * FNB;                        // merges of four weights per substep
    static constexpr int MQS = MF / NMQ;                       // slots between them
    static constexpr int DQS = MF / XG;                        // slots between token loads
    static_assert(FNB <= 2 && FMB > LEAD && MF % NMQ == 0 && MF % XG == 0 && MQS >= 2, "slot plan");
    typedef __attribute__((address_space(3))) uint8_t lds_byte;

    // one K-tile of the wave's weights: 16 bytes of each plane, or the two halves of a packed FP16 block
    struct Raw { u32x4 u[FNB], l[FNB]; };

    struct Ctx {
        floatx4 (&acc)[FNB][FMB];
        intx4 (&a)[2][FNB];                                    // merged weight fragments of substeps 0 / 1
        intx4 (&b)[2][FMB];                                    // token fragments (a few are live at a time)
        Raw (&raw)[NRAW];
        __amdgpu_buffer_rsrc_t rx, rw0, rw1;
        uint32_t x_off, x_step, x_kpos, x_lim;               // offset of the wave's first load, step between its loads
        uint32_t w_off, w_istep, w_kpos, w_lim;              // lane + wave part, step between row tiles, column test
        const uint8_t *lds;
        lds_byte *lds3;
        int wave, lane;
        int kt, st;                                            // K-tile, its LDS stage
        const Regroup<false> &rg;                              // PAIR
    };

    template <int J>
    static __device__ __forceinline__ void read_b(intx4 &dst, const uint8_t *stage, int lane, int s) {
        dst = *reinterpret_cast<const intx4 *>(stage + swz(16 * J + (lane & 15), 4 * s + (lane >> 4)));
    }

    // the lane's columns of K-tile kt lie inside K (w_kpos = 16 (l / 16) for row-major planes, whose
    // rows have no padding; 0 for packed blocks, which are zero-padded to whole blocks); otherwise
    // the load is sent out of the buffer's range and returns zero
    static __device__ __forceinline__ void load_raw(Raw &r, const Ctx &c, int kt) {
        const uint32_t kill = ((uint32_t)kt * 64u + c.w_kpos < c.w_lim) ? 0u : 0x80000000u;
#pragma unroll
        for (int i = 0; i < FNB; ++i) {
            const uint32_t off = (c.w_off + (uint32_t)i * c.w_istep + (uint32_t)kt * (ROWMAJOR ? 64u : (uint32_t)BLOCK_BYTES)) | kill;
            r.u[i] = __builtin_amdgcn_raw_buffer_load_b128(c.rw0, off, 0, POLICY);
            if (MERGE) r.l[i] = __builtin_amdgcn_raw_buffer_load_b128(c.rw1, off, 0, POLICY);
            else r.l[i] = __builtin_amdgcn_raw_buffer_load_b128(c.rw0, off + 1024u, 0, POLICY);
        }
    }

    // PAIR: both planes of K-tiles kt and kt + 1 in load order, rows 0 .. 7 of a tile in r0, 8 .. 15 in r1
    static __device__ __forceinline__ void load_pair(Raw &r0, Raw &r1, const Ctx &c, int kt) {
        const uint32_t kill = ((uint32_t)kt * 64u + c.w_kpos < c.w_lim) ? 0u : 0x80000000u;
        const uint32_t half = c.w_istep >> 1;                  // 8 rows
#pragma unroll
        for (int i = 0; i < FNB; ++i) {
            const uint32_t off = (c.w_off + (uint32_t)i * c.w_istep + (uint32_t)kt * 64u) | kill;
            r0.u[i] = __builtin_amdgcn_raw_buffer_load_b128(c.rw0, off, 0, POLICY);
            r1.u[i] = __builtin_amdgcn_raw_buffer_load_b128(c.rw0, off + half, 0, POLICY);
            r0.l[i] = __builtin_amdgcn_raw_buffer_load_b128(c.rw1, off, 0, POLICY);
            r1.l[i] = __builtin_amdgcn_raw_buffer_load_b128(c.rw1, off + half, 0, POLICY);
        }
    }

    // ... and into operand order, r0 for K-tile kt and r1 for kt + 1; J: row tile and plane
    template <int J>
    static __device__ __forceinline__ void regroup(Raw &r0, Raw &r1, const Ctx &c) {
        if constexpr (J < FNB) c.rg.run(r0.u[J], r1.u[J]);
        else c.rg.run(r0.l[J - FNB], r1.l[J - FNB]);
    }

    // four weights of row tile I: dwords H (substep 0) or 2 + H (substep 1) of the lane's chunk of
    // each plane; packed FP16 weights are taken as they are (first half block = substep 0)
    template <int S, int I, int H>
    static __device__ __forceinline__ void merge_part(intx4 &dst, const Raw &r) {
        if constexpr (MERGE) {
            uint32_t w01, w23;
            merge4(r.u[I][2 * S + H], r.l[I][2 * S + H], w01, w23);
            dst[2 * H] = (int)w01;
            dst[2 * H + 1] = (int)w23;
        } else {
            dst[2 * H] = (int)(S == 0 ? r.u[I][2 * H] : r.l[I][2 * H]);
            dst[2 * H + 1] = (int)(S == 0 ? r.u[I][2 * H + 1] : r.l[I][2 * H + 1]);
        }
    }

    static __device__ __forceinline__ void dma_x(const Ctx &c, int i, int kt) {
        const uint32_t kb = (uint32_t)kt * 128u;
        const uint32_t kill = (kb + c.x_kpos < c.x_lim) ? 0u : 0x80000000u;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(c.rx, (__attribute__((address_space(3))) void *)(c.lds3 + (kt & (NST - 1)) * STAGE + (i * DW + c.wave) * 1024),
                                                 16, (c.x_off + (uint32_t)i * c.x_step + kb) | kill, 0, 0, 0);
    }

    // PAR: which register set holds the plane blocks of this K-tile (the one after it holds the next)
    template <bool OLDER, int S, int PAR, int Q>
    static __device__ __forceinline__ void slot(Ctx &c) {
        constexpr int j = Q / FNB, i = Q % FNB;
        {
            union { intx4 v; half8 h; } a, b;
            a.v = c.a[S][i];
            b.v = c.b[S][j];
            c.acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a.h, b.h, c.acc[i][j], 0, 0, 0);
        }
        if constexpr (i == 0) {
            // token fragment LEAD blocks ahead: this substep, the next one, or the next K-tile
            if constexpr (j + LEAD < FMB) read_b<j + LEAD>(c.b[S][j + LEAD], c.lds + c.st * STAGE, c.lane, S);
            else if constexpr (S == 0) read_b<j + LEAD - FMB>(c.b[1][j + LEAD - FMB], c.lds + c.st * STAGE, c.lane, 1);
            else read_b<j + LEAD - FMB>(c.b[0][j + LEAD - FMB], c.lds + ((c.st + 1) & (NST - 1)) * STAGE, c.lane, 0);
        }
        if constexpr (Q % MQS == MQS - 1) {
            // substep 0 merges this K-tile's second half, substep 1 the next K-tile's first half
            constexpr int m = Q / MQS;
            if constexpr (S == 0) merge_part<1, m / 2, m % 2>(c.a[1][m / 2], c.raw[PAR]);
            else merge_part<0, m / 2, m % 2>(c.a[0][m / 2], c.raw[(PAR + 1) % NRAW]);
        }
        if constexpr (OLDER && S == 0 && Q % DQS == 0) dma_x(c, Q / DQS, c.kt + XA);
        if constexpr (!PAIR) {
            if constexpr (S == 1 && Q == 0) load_raw(c.raw[PAR], c, c.kt + NRAW);  // its blocks are merged
        } else if constexpr (PAR % 2 == 1) {
            // second K-tile of a pair: the next pair has landed, this one is merged
            if constexpr (S == 0 && Q % RGS == 0 && Q / RGS < 2 * FNB) regroup<Q / RGS>(c.raw[(PAR + 1) % NRAW], c.raw[(PAR + 2) % NRAW], c);
            if constexpr (S == 1 && Q == 0) load_pair(c.raw[PAR - 1], c.raw[PAR], c, c.kt - 1 + NRAW);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (Q + 1 < MF) slot<OLDER, S, PAR, Q + 1>(c);
    }

    template <bool OLDER, int PAR>
    static __device__ __forceinline__ void k_tile(Ctx &c) {
        __builtin_amdgcn_sched_barrier(0);
        slot<OLDER, 0, PAR, 0>(c);
        slot<OLDER, 1, PAR, 0>(c);
        // The token loads of K-tile kt+2 (issued during kt+2-XA) must have landed before anybody
        // reads them (from the tail of kt+1 on).  Younger than them in this wave, and allowed to
        // be in flight: the plane loads of that K-tile and all loads of the XA-2 K-tiles since
        // (for XA = 3 the count is rounded down to this K-tile's loads).  PAIR: 4 FNB plane loads at the end of
        // every second K-tile, which fall on XA / 2 of the XA - 1 K-tiles since, or one less.
        constexpr int kInFlight = PAIR ? (XA - 2) * XG + ((XA - 1 + (PAR & 1)) / 2) * 4 * FNB
                                       : (XA == 3 ? XG + 2 * FNB : 2 * FNB + (XA - 2) * (XG + 2 * FNB));
        if constexpr (OLDER) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kInFlight) : "memory");
        // a bare barrier: __syncthreads() carries a release fence, which would drain the token loads
        // issued in this K-tile.  What the fence would order is ordered by the wait above (loads
        // that have to be visible) and by the MFMAs, which have consumed every LDS read of the
        // stage that is refilled next.
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }

    template <bool OLDER>
    static __device__ __forceinline__ void k_loop(Ctx &c, int kt_begin, int kt_end) {
        // no branch inside the loop body: the compiler then counts the loads in flight exactly
        // instead of draining them at the loop head
        int kt = kt_begin;
        if constexpr (PAIR) {
            // whole pairs: the second K-tile of the last one may lie past the slice, where tokens and weights
            // are zero.  (A tail of 1 .. 3 single K-tiles cost registers that the loop spilled.)
            for (; kt + NRAW - 2 < kt_end; kt += NRAW) k_tiles<OLDER, 0, NRAW>(c, kt);
            pair_tail<OLDER, 0>(c, kt, kt_end);
        } else {
            for (; kt + NRAW <= kt_end; kt += NRAW) k_tiles<OLDER, 0, NRAW>(c, kt);
            tail<OLDER, 0>(c, kt, kt_end);
        }
    }

    // K-tiles kt + P .. kt + END - 1, on register sets P .. END - 1
    template <bool OLDER, int P, int END>
    static __device__ __forceinline__ void k_tiles(Ctx &c, int kt) {
        c.kt = kt + P;
        c.st = (kt + P) & (NST - 1);
        k_tile<OLDER, P>(c);
        if constexpr (P + 1 < END) k_tiles<OLDER, P + 1, END>(c, kt);
    }

    // the last 0 .. NRAW / 2 - 1 pairs
    template <bool OLDER, int P>
    static __device__ __forceinline__ void pair_tail(Ctx &c, int kt, int kt_end) {
        if constexpr (P + 2 < NRAW) {
            if (kt + P < kt_end) {
                k_tiles<OLDER, P, P + 2>(c, kt);
                pair_tail<OLDER, P + 2>(c, kt, kt_end);
            }
        }
    }

    // the last 0 .. NRAW - 1 K-tiles (not PAIR)
    template <bool OLDER, int P>
    static __device__ __forceinline__ void tail(Ctx &c, int kt, int kt_end) {
        if constexpr (P + 1 < NRAW) {
            if (kt + P < kt_end) {
                k_tiles<OLDER, P, P + 1>(c, kt);
                tail<OLDER, P + 1>(c, kt, kt_end);
            }
        }
    }

    static __device__ __forceinline__ void run(const LargeParams &p, uint8_t *lds, lds_byte *lds3) {
        const int lane = threadIdx.x & 63;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        int tm, tn;
        tile_of_block(p, blockIdx.x, tm, tn);
        const int m0 = tm * TM, n0 = tn * TN;
        const int split = blockIdx.y;
        // the LDS stage of a K-tile is kt % 4: start the slice on a multiple of 4 as far as the ring goes
        const int kt_begin = split * p.ktiles_per_split;
        const int kt_end = min(kt_begin + p.ktiles_per_split, p.ktiles_total);

        floatx4 acc[FNB][FMB];
#pragma unroll
        for (int i = 0; i < FNB; ++i)
#pragma unroll
            for (int j = 0; j < FMB; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
        intx4 a[2][FNB], b[2][FMB];
        Raw raw[NRAW];
        const Regroup<false> rg(lds, (uint32_t)(RING_BYTES + wave * 2048), lane);
        const int w_rows = min(TN, p.N - n0);
        Ctx c{acc, a, b, raw,
              tile_rsrc(p.X, m0, min(TM, p.M - m0), p.x_row_bytes, p.k_bytes),
              ROWMAJOR ? tile_rsrc(p.W0, n0, w_rows, p.w_row_bytes, p.K) : plane_rsrc(p.W0, n0, w_rows, p.kblocks, BLOCK_BYTES),
              ROWMAJOR ? tile_rsrc(p.W1, n0, w_rows, p.w_row_bytes, p.K)
                       : plane_rsrc(MERGE ? p.W1 : p.W0, n0, w_rows, p.kblocks, BLOCK_BYTES),
              0u, (uint32_t)(DW * 8) * (uint32_t)p.x_row_bytes, 0u, slice_end(p, kt_end), 0u, 0u, 0u, 0u, lds, lds3, wave, lane,
              kt_begin, 0, rg};
        {
            const int pc = lane & 7;
            const int ch = fp16_chunk_of_slot(pc ^ ((((wave & 1) << 2) + (lane >> 4)) & 7));   // (row >> 1) & 7 for row = gid*8 + lane/8
            c.x_kpos = 16u * ch;
            c.x_off = (uint32_t)(wave * 8 + (lane >> 3)) * (uint32_t)p.x_row_bytes + 16u * ch;
            if (ROWMAJOR) {
                const uint32_t row = PAIR ? lane >> 3 : lane & 15, chunk = PAIR ? lane & 7 : lane >> 4;
                c.w_off = (uint32_t)(FNB * wave * 16 + row) * (uint32_t)p.w_row_bytes + 16u * chunk;
                c.w_istep = 16u * (uint32_t)p.w_row_bytes;
                c.w_kpos = 16u * chunk;
                c.w_lim = slice_end(p, kt_end) >> 1;
            } else {
                c.w_off = (uint32_t)(FNB * wave * p.kblocks) * (uint32_t)BLOCK_BYTES + (uint32_t)lane * 16u;
                c.w_istep = (uint32_t)p.kblocks * (uint32_t)BLOCK_BYTES;
                c.w_kpos = 0u;
                c.w_lim = (uint32_t)min(p.kblocks, kt_end) * 64u;
            }
        }
        // token tiles of the first XA K-tiles, plane blocks of the first NRAW
        if (wave < DW) {
#pragma unroll
            for (int d = 0; d < XA; ++d)
#pragma unroll
                for (int i = 0; i < XG; ++i) dma_x(c, i, kt_begin + d);
        }
#pragma unroll
        for (int d = 0; d < NRAW; ++d) {
            if constexpr (!PAIR) load_raw(raw[d], c, kt_begin + d);
            else if (d % 2 == 0) load_pair(raw[d], raw[d + 1], c, kt_begin + d);
        }
        // (in order: once the first plane blocks are here, the token loads issued before them are too)
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PAIR ? 4 * FNB : (NRAW - 1) * 2 * FNB) : "memory");
        if constexpr (PAIR) {
            regroup<0>(raw[0], raw[1], c);
            regroup<1>(raw[0], raw[1], c);
            if constexpr (FNB > 1) {
                regroup<2>(raw[0], raw[1], c);
                regroup<3>(raw[0], raw[1], c);
            }
        }
        merge_part<0, 0, 0>(a[0][0], raw[0]);
        merge_part<0, 0, 1>(a[0][0], raw[0]);
        if constexpr (FNB > 1) {
            merge_part<0, FNB - 1, 0>(a[0][FNB - 1], raw[0]);
            merge_part<0, FNB - 1, 1>(a[0][FNB - 1], raw[0]);
        }
        // (a bare barrier, as in the loop: the later plane loads stay in flight)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        c.st = kt_begin & (NST - 1);
        {
            const uint8_t *st0 = lds + c.st * STAGE;
            read_b<0>(b[0][0], st0, lane, 0);
            if (LEAD > 1) read_b<1>(b[0][1], st0, lane, 0);
            if (LEAD > 2) read_b<2>(b[0][2], st0, lane, 0);
            if (LEAD > 3) read_b<3>(b[0][3], st0, lane, 0);
        }
        if (wave < DW) k_loop<true>(c, kt_begin, kt_end);
        else k_loop<false>(c, kt_begin, kt_end);
        // token loads of K-tiles past the end are still in flight: they must have landed before the
        // LDS is reused for the output tile or handed back
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        // (keeps the epilogue's address arithmetic behind the loop, where registers are free)
        int lane_out = lane;
        asm volatile("" : "+v"(lane_out));
        if (gridDim.y == 1) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the look-ahead fragment reads
            __syncthreads();
            Store::epilogue_lds(p, acc, m0, n0, 0, wave, lane_out, wave, lds);
        } else {
            Store::store_partials(p, acc, m0, n0, 0, wave, lane_out, split);
        }
    }
};

template <int TM, int TN, int WK, bool DEEP, bool NT, bool PAIRS>
__global__ void __launch_bounds__(512)
nested_bypass_kernel(LargeParams p) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
    typedef BypassKernel<TM, TN, WK, DEEP, NT, PAIRS> Kern;
    Kern::run(p, lds_raw, (typename Kern::lds_byte *)lds_raw);
}

// ---- NestedFP16 from row-major planes, by pairs of K-tiles ------------------------------------------
// The same layout of work as nested_bypass_kernel, but the planes reach their wave through LDS: both planes
// of two K-tiles are copied there directly, 128 bytes of 8 rows per instruction, into a part of the LDS that
// only this wave uses (4 KB for 16 weight rows), and a lane reads its 16 bytes of each plane from there one
// K-tile before they are merged.  Loaded straight into registers in operand order, 16 rows x 64 bytes per
// instruction, every 128-byte line is requested twice: a load-only kernel takes in 38 bytes per nanosecond
// and CU so, and 137 by whole lines.
// (28672, 4096): 100 tokens 61.8 us with pairs regrouped in registers, 56.5 so; 2048 tokens 452 us in operand order, 435 so;
// 128 x 256 tiles gain 12-28 %.
// A pair's copies are under way while the pair before it is multiplied from registers (1.7 K-tiles).  The
// one barrier of a K-tile sits behind the last read of its token stage, in the last slots of the second
// substep: the next K-tile's tokens have to be there by then, and the stage is free from then on, so that
// three stages give the token copies two K-tiles.
template <int TM, int TN, bool NT>
struct RowsKernel {
    typedef TileStore<kNestedF16, TM, TN, 1, 8> Store;
    static constexpr int DW = 4;                               // waves that issue the token copies
    static constexpr int WTN = TN / 8;
    static constexpr int FMB = TM / 16, FNB = WTN / 16;
    static constexpr int MF = FMB * FNB;                       // MFMAs per substep
    static constexpr int NST = TM > 192 ? 3 : 4;               // LDS stages of the token tile
    static constexpr int XA = NST - 1;                         // token copies run this many K-tiles ahead
    static constexpr int STAGE = TM * 128;
    static constexpr int OWN = FNB * 4096;                     // both planes of a pair of K-tiles of the wave's rows
    static constexpr int RING_BYTES = NST * STAGE;
    static constexpr int LDS_BYTES = RING_BYTES + 8 * OWN > TM * TN * 2 ? RING_BYTES + 8 * OWN : TM * TN * 2;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS");
    static constexpr int POLICY = NT ? 2 : 0;                  // see BypassKernel
    static constexpr int XG = TM / 8 / DW;                     // token copies per loading wave and K-tile
    static constexpr int WG = 4 * FNB;                         // weight copies per wave and pair
    static constexpr int LEAD = 2;                             // token fragments are read this many blocks ahead
    static constexpr int NMQ = 2 * FNB;                        // merges of four weights per substep
    static constexpr int MQS = MF / NMQ;                       // slots between them
    static constexpr int DQS = MF / XG;                        // slots between token copies
    static constexpr int QB = MF - 2;                          // slot that starts with the barrier
    // Second substep of a pair's second K-tile: the next pair's bytes are read in slots 0 .. 2 FNB - 1, two per slot,
    // and the copies of the pair after it are issued from slot QW on, all before the barrier and spread out: bunched in
    // consecutive slots, where every wave waits for the address queue, they cost 1.5 % at 256 x 256.
    static constexpr int QW = 2 * FNB + 2;
    static constexpr int WPS = (WG + (QB - QW) - 1) / (QB - QW);         // copies per slot that issues any
    static constexpr int WSTR = WG <= QB - QW ? (QB - QW) / WG : 1;      // slots between them
    static_assert(FNB <= 2 && FMB > LEAD && MF % NMQ == 0 && MF % XG == 0 && MQS >= 2 && QW > 2 * FNB && QB > QW, "slot plan");
    typedef __attribute__((address_space(3))) uint8_t lds_byte;

    struct Raw { u32x4 u[FNB], l[FNB]; };                      // one K-tile of the wave's weights: 16 bytes of each plane

    struct Ctx {
        floatx4 (&acc)[FNB][FMB];
        intx4 (&a)[2][FNB];                                    // merged weight fragments of substeps 0 / 1
        intx4 (&b)[2][FMB];                                    // token fragments (a few are live at a time)
        Raw (&raw)[2];                                         // first and second K-tile of a pair
        __amdgpu_buffer_rsrc_t rx, rw0, rw1;
        uint32_t x_off, x_step, x_kpos, x_lim;                 // offset of the wave's first token copy, step between its copies
        uint32_t w_off, w_step, w_kpos, w_lim;                 // rows 0 .. 7; step to rows 8 .. 15; column; end of the slice
        uint32_t own, get;                                     // LDS: the wave's part, the lane's chunk of the first K-tile
        uint8_t *lds;
        lds_byte *lds3;
        int wave, lane;
        int kt, st, fill;                                      // K-tile, its LDS stage, the stage that is filled
    };

    static __device__ __forceinline__ int next(int st) { return st + 1 == NST ? 0 : st + 1; }

    template <int J>
    static __device__ __forceinline__ void read_b(intx4 &dst, const uint8_t *stage, int lane, int s) {
        dst = *reinterpret_cast<const intx4 *>(stage + swz(16 * J + (lane & 15), 4 * s + (lane >> 4)));
    }

    // piece D (row tile D / 2; upper plane, lower plane) of a pair's first (P = 0) or second K-tile: chunk g or 4 + g of
    // the lane's row, whose place differs in one bit
    template <int P, int D>
    static __device__ __forceinline__ void read_raw(Raw &r, const Ctx &c) {
        const u32x4 v = *reinterpret_cast<const u32x4 *>(c.lds + (P == 0 ? c.get : c.get ^ 64u) + D * 2048);
        if constexpr (D % 2 == 0) r.u[D / 2] = v;
        else r.l[D / 2] = v;
    }
    template <int D>
    static __device__ __forceinline__ void read_pair(const Ctx &c) {     // D of 4 FNB
        if constexpr (D < 2 * FNB) read_raw<0, D>(c.raw[0], c);
        else read_raw<1, D - 2 * FNB>(c.raw[1], c);
    }
    // the bytes read above have arrived: from here on their place may be written
    static __device__ __forceinline__ void have_pair(const Ctx &c) {
#pragma unroll
        for (int i = 0; i < FNB; ++i) {
            asm volatile("" : "+v"(c.raw[0].u[i]), "+v"(c.raw[0].l[i]) :: "memory");
            asm volatile("" : "+v"(c.raw[1].u[i]), "+v"(c.raw[1].l[i]) :: "memory");
        }
    }

    // copy D of a pair that starts with K-tile kt: row tile D / 4, plane D / 2 % 2, rows 0 .. 7 or 8 .. 15; a chunk past
    // the slice is sent out of range and arrives as zeros
    static __device__ __forceinline__ void dma_w(const Ctx &c, int d, int kt) {
        const uint32_t flip = (uint32_t)(d & 1) << 6;          // rows 8 .. 15 swizzle with the top bit set
        const uint32_t col = (uint32_t)kt * 64u + (c.w_kpos ^ flip);
        const uint32_t kill = col < c.w_lim ? 0u : 0x80000000u;
        const uint32_t off = (c.w_off + (uint32_t)(2 * (d >> 2) + (d & 1)) * c.w_step + col) | kill;
        __builtin_amdgcn_raw_ptr_buffer_load_lds((d & 2) ? c.rw1 : c.rw0,
            (__attribute__((address_space(3))) void *)(c.lds3 + c.own + (uint32_t)((d >> 1) * 2048 + (d & 1) * 1024)), 16, off, 0, 0, POLICY);
    }

    static __device__ __forceinline__ void dma_x(const Ctx &c, int i, int kt, int stage) {
        const uint32_t kb = (uint32_t)kt * 128u;
        const uint32_t kill = (kb + c.x_kpos < c.x_lim) ? 0u : 0x80000000u;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(c.rx, (__attribute__((address_space(3))) void *)(c.lds3 + stage * STAGE + (i * DW + c.wave) * 1024),
                                                 16, (c.x_off + (uint32_t)i * c.x_step + kb) | kill, 0, 0, 0);
    }

    // four weights of row tile I: dwords H (substep 0) or 2 + H (substep 1) of the lane's chunk of each plane
    template <int S, int I, int H>
    static __device__ __forceinline__ void merge_part(intx4 &dst, const Raw &r) {
        uint32_t w01, w23;
        merge4(r.u[I][2 * S + H], r.l[I][2 * S + H], w01, w23);
        dst[2 * H] = (int)w01;
        dst[2 * H + 1] = (int)w23;
    }

    // PAR: first or second K-tile of a pair.  OLDER: one of the DW waves that copy tokens.
    template <bool OLDER, int S, int PAR, int Q>
    static __device__ __forceinline__ void slot(Ctx &c) {
        constexpr int j = Q / FNB, i = Q % FNB;
        if constexpr (S == 1 && Q == QB) {
            // the last fragments of this stage have arrived, and the next K-tile's tokens have landed.  Younger than
            // those in a loading wave: the tokens of the XA - 1 K-tiles after it and the weights copied in the
            // XA K-tiles since.
            asm volatile("" : "+v"(c.b[1][FMB - 1]), "+v"(c.b[1][FMB - 2]));
            if constexpr (OLDER) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((XA - 1) * XG + (XA + PAR) / 2 * WG) : "memory");
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (S == 1 && PAR == 1) {
            if constexpr (Q == 0) {
                // the next pair has landed (this wave's own copies; younger: the tokens of two K-tiles)
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(OLDER ? 2 * XG : 0) : "memory");
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (Q == QW) {
                have_pair(c);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        {
            union { intx4 v; half8 h; } a, b;
            a.v = c.a[S][i];
            b.v = c.b[S][j];
            c.acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a.h, b.h, c.acc[i][j], 0, 0, 0);
        }
        // token fragments LEAD blocks ahead: this substep, the next one; those of the next K-tile behind the barrier
        if constexpr (i == 0) {
            if constexpr (j + LEAD < FMB) read_b<j + LEAD>(c.b[S][j + LEAD], c.lds + c.st * STAGE, c.lane, S);
            else if constexpr (S == 0) read_b<j + LEAD - FMB>(c.b[1][j + LEAD - FMB], c.lds + c.st * STAGE, c.lane, 1);
        }
        if constexpr (S == 1 && Q >= QB) read_b<Q - QB>(c.b[0][Q - QB], c.lds + next(c.st) * STAGE, c.lane, 0);
        if constexpr (S == 1 && PAR == 1) {
            if constexpr (Q < 2 * FNB) {
                read_pair<2 * Q>(c);
                read_pair<2 * Q + 1>(c);
            }
            if constexpr (Q >= QW && Q < QB && (Q - QW) % WSTR == 0) {
#pragma unroll
                for (int d = (Q - QW) / WSTR * WPS; d < ((Q - QW) / WSTR + 1) * WPS && d < WG; ++d) dma_w(c, d, c.kt + 3);
            }
        }
        if constexpr (Q % MQS == MQS - 1) {
            // substep 0 merges this K-tile's second half, substep 1 the next K-tile's first half
            constexpr int m = Q / MQS;
            if constexpr (S == 0) merge_part<1, m / 2, m % 2>(c.a[1][m / 2], c.raw[PAR]);
            else merge_part<0, m / 2, m % 2>(c.a[0][m / 2], c.raw[PAR ^ 1]);
        }
        if constexpr (OLDER && S == 0 && Q % DQS == 0) dma_x(c, Q / DQS, c.kt + XA, c.fill);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (Q + 1 < MF) slot<OLDER, S, PAR, Q + 1>(c);
    }

    template <bool OLDER, int PAR>
    static __device__ __forceinline__ void k_tile(Ctx &c, int kt) {
        c.kt = kt;
        __builtin_amdgcn_sched_barrier(0);
        slot<OLDER, 0, PAR, 0>(c);
        slot<OLDER, 1, PAR, 0>(c);
        c.fill = c.st;
        c.st = next(c.st);
    }

    // whole pairs: the second K-tile of the last one may lie past the slice, where tokens and weights are zero
    template <bool OLDER>
    static __device__ __forceinline__ void k_loop(Ctx &c, int kt_begin, int kt_end) {
        for (int kt = kt_begin; kt < kt_end; kt += 2) {
            k_tile<OLDER, 0>(c, kt);
            k_tile<OLDER, 1>(c, kt + 1);
        }
    }

    static __device__ __forceinline__ void run(const LargeParams &p, uint8_t *lds, lds_byte *lds3) {
        const int lane = threadIdx.x & 63;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        int tm, tn;
        tile_of_block(p, blockIdx.x, tm, tn);
        const int m0 = tm * TM, n0 = tn * TN;
        const int split = blockIdx.y;
        const int kt_begin = split * p.ktiles_per_split;
        const int kt_end = min(kt_begin + p.ktiles_per_split, p.ktiles_total);

        floatx4 acc[FNB][FMB];
#pragma unroll
        for (int i = 0; i < FNB; ++i)
#pragma unroll
            for (int j = 0; j < FMB; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
        intx4 a[2][FNB], b[2][FMB];
        Raw raw[2];
        const int w_rows = min(TN, p.N - n0);
        const uint32_t own = (uint32_t)(RING_BYTES + wave * OWN);
        const int r16 = lane & 15, g = lane >> 4;
        const int xch = fp16_chunk_of_slot((lane & 7) ^ ((((wave & 1) << 2) + g) & 7));      // (row >> 1) & 7 for row = 8 (4 i + wave) + lane / 8
        Ctx c{acc, a, b, raw,
              tile_rsrc(p.X, m0, min(TM, p.M - m0), p.x_row_bytes, p.k_bytes),
              tile_rsrc(p.W0, n0, w_rows, p.w_row_bytes, p.K), tile_rsrc(p.W1, n0, w_rows, p.w_row_bytes, p.K),
              (uint32_t)(wave * 8 + (lane >> 3)) * (uint32_t)p.x_row_bytes + 16u * xch, (uint32_t)(DW * 8) * (uint32_t)p.x_row_bytes,
              16u * xch, slice_end(p, kt_end),
              (uint32_t)(FNB * wave * 16 + (lane >> 3)) * (uint32_t)p.w_row_bytes, 8u * (uint32_t)p.w_row_bytes,
              16u * (uint32_t)((lane & 7) ^ g), slice_end(p, kt_end) >> 1,                  // (rows 0 .. 7: (row >> 1) & 7 = lane / 16)
              own, own + (uint32_t)r16 * 128u + (uint32_t)((g ^ (r16 >> 1)) << 4),
              lds, lds3, wave, lane, kt_begin, 0, XA};
        // the first pair of the weights, the first XA K-tiles of the tokens
#pragma unroll
        for (int d = 0; d < WG; ++d) dma_w(c, d, kt_begin);
        if (wave < DW) {
#pragma unroll
            for (int d = 0; d < XA; ++d)
#pragma unroll
                for (int i = 0; i < XG; ++i) dma_x(c, i, kt_begin + d, d);
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((XA - 1) * XG) : "memory");
        } else {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        read_pair<0>(c);
        read_pair<1>(c);
        read_pair<2>(c);
        read_pair<3>(c);
        if constexpr (FNB > 1) {
            read_pair<4>(c);
            read_pair<5>(c);
            read_pair<6>(c);
            read_pair<7>(c);
        }
        read_b<0>(b[0][0], lds, lane, 0);
        read_b<1>(b[0][1], lds, lane, 0);
        have_pair(c);
        // (its copies are the youngest before the loop, as those of any later pair are when the next K-tile begins)
#pragma unroll
        for (int d = 0; d < WG; ++d) dma_w(c, d, kt_begin + 2);
        merge_part<0, 0, 0>(a[0][0], raw[0]);
        merge_part<0, 0, 1>(a[0][0], raw[0]);
        if constexpr (FNB > 1) {
            merge_part<0, FNB - 1, 0>(a[0][FNB - 1], raw[0]);
            merge_part<0, FNB - 1, 1>(a[0][FNB - 1], raw[0]);
        }
        if (wave < DW) k_loop<true>(c, kt_begin, kt_end);
        else k_loop<false>(c, kt_begin, kt_end);
        // copies of K-tiles past the end are still in flight: they must have landed before the LDS is reused
        // for the output tile or handed back
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        // (keeps the epilogue's address arithmetic behind the loop, where registers are free)
        int lane_out = lane;
        asm volatile("" : "+v"(lane_out));
        if (gridDim.y == 1) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the look-ahead fragment reads
            __syncthreads();
            Store::epilogue_lds(p, acc, m0, n0, 0, wave, lane_out, wave, lds);
        } else {
            Store::store_partials(p, acc, m0, n0, 0, wave, lane_out, split);
        }
    }
};

template <int TM, int TN, bool NT>
__global__ void __launch_bounds__(512)
nested_rows_kernel(LargeParams p) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
    typedef RowsKernel<TM, TN, NT> Kern;
    Kern::run(p, lds_raw, (typename Kern::lds_byte *)lds_raw);
}

// ---- FP8 mode on at most 64 tokens per tile: E4M3 weights through registers ---------------------
// The same layout of work as nested_bypass_kernel (eight waves side by side along the weight rows,
// packed 1 KB blocks loaded 16 bytes per lane, token tile in a ring of four LDS stages), for
// batches where the weight stream is the bound.  A K-tile is 128 bytes of a token row and two
// blocks of the upper plane; lane group g = l / 16 holds columns 16 g .. + 15 of both blocks, 32
// bytes, which is one operand of v_mfma_f32_16x16x128_f8f6f4, and reads the same bytes of its token
// (chunks g and 4 + g of the row).  A token block's fragment of K-tile kt + 1 is read right behind
// the block's MFMAs of K-tile kt, into the same registers.
// Row-major planes: a K-tile's 128 bytes of 16 rows are fetched as 128 bytes of 8 rows per instruction and
// regrouped through 2 KB of LDS per wave during the K-tile before (see Regroup); NT: the rows start on
// lines, which are then read once and marked non-temporal.
template <int TM, int TN, bool ROWMAJOR, bool NT = false>
struct E4m3BypassKernel {
    typedef TileStore<kE4M3, TM, TN, 1, 8, 16> Store;
    static constexpr int DW = 4;                               // waves that issue the token loads
    static constexpr int WTN = TN / 8;
    static constexpr int FMB = TM / 16, FNB = WTN / 16;
    static constexpr int NST = 8;                              // LDS stages of the token tile
    static constexpr int XA = 6;                               // token loads run this many K-tiles ahead
    static constexpr int NRAW = 4;                             // plane blocks are loaded this many K-tiles ahead
    static constexpr int STAGE = TM * 128;
    static constexpr int RING_BYTES = NST * STAGE > TM * TN * 2 ? NST * STAGE : TM * TN * 2;
    static constexpr int LDS_BYTES = RING_BYTES + (ROWMAJOR ? 8 * 2048 : 0);
    static constexpr int XG = TM / 8 / DW;                     // loads per loading wave per K-tile
    static_assert(XG >= 1 && FNB >= 1 && FNB <= 2, "tile shape");
    static_assert(XA >= 3 && XA < NST && NRAW <= XA, "the stage being filled is neither the one in use nor the next");
    typedef __attribute__((address_space(3))) uint8_t lds_byte;

    static constexpr int POLICY = NT ? 2 : 0;                  // whole lines, read once per launch: non-temporal
    struct Raw { intx4 u[FNB][2]; };                           // one K-tile of the wave's plane blocks
    struct Tok { intx4 q[FMB][2]; };                           // one K-tile of token fragments

    struct Ctx {
        floatx4 (&acc)[FNB][FMB];
        Raw (&raw)[NRAW];
        Tok &tok;                                              // block J is re-read for the next K-tile right behind its MFMAs
        __amdgpu_buffer_rsrc_t rx, rw;
        uint32_t x_off, x_step, x_kpos, x_lim;
        uint32_t w_off, w_istep, w_kpos, w_lim;              // as in the NestedFP16 kernel
        const uint8_t *lds;
        lds_byte *lds3;
        int wave, lane;
        int kt;
        const Regroup<false> &rg;                              // row-major planes
    };

    // row-major: rows 0 .. 7 / 8 .. 15 of the 16 into u[i][0] / u[i][1]
    static __device__ __forceinline__ void regroup(Raw &r, const Ctx &c) {
#pragma unroll
        for (int i = 0; i < FNB; ++i) {
            u32x4 a = __builtin_bit_cast(u32x4, r.u[i][0]), b = __builtin_bit_cast(u32x4, r.u[i][1]);
            c.rg.run(a, b);
            r.u[i][0] = __builtin_bit_cast(intx4, a);
            r.u[i][1] = __builtin_bit_cast(intx4, b);
        }
    }

    static __device__ __forceinline__ void load_raw(Raw &r, const Ctx &c, int kt) {
        if constexpr (ROWMAJOR) {
            const uint32_t kill = ((uint32_t)kt * 128u + c.w_kpos < c.w_lim) ? 0u : 0x80000000u;
#pragma unroll
            for (int i = 0; i < FNB; ++i) {
                const uint32_t off = (c.w_off + (uint32_t)i * c.w_istep + (uint32_t)kt * 128u) | kill;
                r.u[i][0] = __builtin_bit_cast(intx4, __builtin_amdgcn_raw_buffer_load_b128(c.rw, off, 0, POLICY));
                r.u[i][1] = __builtin_bit_cast(intx4, __builtin_amdgcn_raw_buffer_load_b128(c.rw, off + (c.w_istep >> 1), 0, POLICY));
            }
            return;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t kill = ((uint32_t)(2 * kt + h) * 64u + c.w_kpos < c.w_lim) ? 0u : 0x80000000u;
#pragma unroll
            for (int i = 0; i < FNB; ++i)
                r.u[i][h] = __builtin_bit_cast(intx4, __builtin_amdgcn_raw_buffer_load_b128(
                    c.rw, (c.w_off + (uint32_t)i * c.w_istep + (uint32_t)(2 * kt + h) * 1024u) | kill, 0, POLICY));
        }
    }

    static __device__ __forceinline__ void dma_x(const Ctx &c, int i, int kt) {
        const uint32_t kb = (uint32_t)kt * 128u;
        const uint32_t kill = (kb + c.x_kpos < c.x_lim) ? 0u : 0x80000000u;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(c.rx, (__attribute__((address_space(3))) void *)(c.lds3 + (kt & (NST - 1)) * STAGE + (i * DW + c.wave) * 1024),
                                                 16, (c.x_off + (uint32_t)i * c.x_step + kb) | kill, 0, 0, 0);
    }

    template <int J>
    static __device__ __forceinline__ void read_tok(Tok &t, const uint8_t *stage, int lane) {
        t.q[J][0] = *reinterpret_cast<const intx4 *>(stage + swz(16 * J + (lane & 15), lane >> 4));
        t.q[J][1] = *reinterpret_cast<const intx4 *>(stage + swz(16 * J + (lane & 15), 4 + (lane >> 4)));
    }

    template <int J>
    static __device__ __forceinline__ void block(Ctx &c, const Raw &r, const uint8_t *next_stage) {
        const intx8 b = __builtin_shufflevector(c.tok.q[J][0], c.tok.q[J][1], 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
        for (int i = 0; i < FNB; ++i) {
            const intx8 a = __builtin_shufflevector(r.u[i][0], r.u[i][1], 0, 1, 2, 3, 4, 5, 6, 7);
            c.acc[i][J] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c.acc[i][J], 0, 0, 0, 0, 0, 0);
        }
        read_tok<J>(c.tok, next_stage, c.lane);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (J + 1 < FMB) block<J + 1>(c, r, next_stage);
    }

    // PAR: which register set holds this K-tile's plane blocks
    template <bool OLDER, int PAR>
    static __device__ __forceinline__ void k_tile(Ctx &c) {
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (OLDER) {
#pragma unroll
            for (int i = 0; i < XG; ++i) dma_x(c, i, c.kt + XA);
        }
        if constexpr (ROWMAJOR) regroup(c.raw[(PAR + 1) % NRAW], c);
        block<0>(c, c.raw[PAR], c.lds + ((c.kt + 1) & (NST - 1)) * STAGE);
        load_raw(c.raw[PAR], c, c.kt + NRAW);                  // its blocks are used up
        // The token loads of K-tile kt+2 (issued during kt+2-XA) must have landed before anybody
        // reads them (during kt+1).  Younger than them in this wave, and allowed to be in flight:
        // the plane loads of that K-tile and all loads of the XA-2 K-tiles since.
        if constexpr (OLDER) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * FNB + (XA - 2) * (XG + 2 * FNB)) : "memory");
        // a bare barrier: __syncthreads() carries a release fence, which would drain the token loads
        // just issued.  What the fence would order is ordered by the wait above (loads that have to
        // be visible) and by the MFMAs that consumed every LDS read of the stage refilled next.
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }

    template <bool OLDER>
    static __device__ __forceinline__ void k_loop(Ctx &c, int kt_begin, int kt_end) {
        static_assert(NRAW == 4, "unrolled by the number of register sets");
        int kt = kt_begin;
        for (; kt + 4 <= kt_end; kt += 4) {
            c.kt = kt;
            k_tile<OLDER, 0>(c);
            c.kt = kt + 1;
            k_tile<OLDER, 1>(c);
            c.kt = kt + 2;
            k_tile<OLDER, 2>(c);
            c.kt = kt + 3;
            k_tile<OLDER, 3>(c);
        }
        if (kt < kt_end) {
            c.kt = kt;
            k_tile<OLDER, 0>(c);
            if (kt + 1 < kt_end) {
                c.kt = kt + 1;
                k_tile<OLDER, 1>(c);
                if (kt + 2 < kt_end) {
                    c.kt = kt + 2;
                    k_tile<OLDER, 2>(c);
                }
            }
        }
    }

    static __device__ __forceinline__ void run(const LargeParams &p, uint8_t *lds, lds_byte *lds3) {
        const int lane = threadIdx.x & 63;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        int tm, tn;
        tile_of_block(p, blockIdx.x, tm, tn);
        const int m0 = tm * TM, n0 = tn * TN;
        const int split = blockIdx.y;
        const int kt_begin = split * p.ktiles_per_split;
        const int kt_end = min(kt_begin + p.ktiles_per_split, p.ktiles_total);

        floatx4 acc[FNB][FMB];
#pragma unroll
        for (int i = 0; i < FNB; ++i)
#pragma unroll
            for (int j = 0; j < FMB; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
        Raw raw[NRAW];
        Tok tok;
        const Regroup<false> rg(lds, (uint32_t)(RING_BYTES + wave * 2048), lane);
        const int w_rows = min(TN, p.N - n0);
        Ctx c{acc, raw, tok,
              tile_rsrc(p.X, m0, min(TM, p.M - m0), p.x_row_bytes, p.k_bytes),
              ROWMAJOR ? tile_rsrc(p.W0, n0, w_rows, p.w_row_bytes, p.K) : plane_rsrc(p.W0, n0, w_rows, p.kblocks, 1024),
              0u, (uint32_t)(DW * 8) * (uint32_t)p.x_row_bytes, 0u, slice_end(p, kt_end), 0u, 0u, 0u, 0u, lds, lds3, wave, lane,
              kt_begin, rg};
        {
            const int ch = (lane & 7) ^ ((((wave & 1) << 2) + (lane >> 4)) & 7);    // (row >> 1) & 7 for row = gid*8 + lane/8
            c.x_kpos = 16u * ch;
            c.x_off = (uint32_t)(wave * 8 + (lane >> 3)) * (uint32_t)p.x_row_bytes + 16u * ch;
            if (ROWMAJOR) {
                c.w_off = (uint32_t)(FNB * wave * 16 + (lane >> 3)) * (uint32_t)p.w_row_bytes + 16u * (uint32_t)(lane & 7);
                c.w_istep = 16u * (uint32_t)p.w_row_bytes;
                c.w_kpos = 16u * (uint32_t)(lane & 7);
                c.w_lim = slice_end(p, kt_end);
            } else {
                c.w_off = (uint32_t)(FNB * wave * p.kblocks) * 1024u + (uint32_t)lane * 16u;
                c.w_istep = (uint32_t)p.kblocks * 1024u;
                c.w_kpos = 0u;
                c.w_lim = (uint32_t)min(p.kblocks, 2 * kt_end) * 64u;
            }
        }
        // token tiles of the first XA K-tiles, plane blocks of the first NRAW
        if (wave < DW) {
#pragma unroll
            for (int d = 0; d < XA; ++d)
#pragma unroll
                for (int i = 0; i < XG; ++i) dma_x(c, i, kt_begin + d);
        }
#pragma unroll
        for (int d = 0; d < NRAW; ++d) load_raw(raw[d], c, kt_begin + d);
        // the token tiles of the first two K-tiles: in order, everything but the later token loads
        // and the plane loads has landed
        if (wave < DW) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((XA - 2) * XG + NRAW * 2 * FNB) : "memory");
        // (a bare barrier, as in the loop: the other loads stay in flight)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if constexpr (ROWMAJOR) regroup(raw[0], c);
        {
            const uint8_t *st0 = lds + (kt_begin & (NST - 1)) * STAGE;
            read_tok<0>(tok, st0, lane);
            if constexpr (FMB > 1) read_tok<1>(tok, st0, lane);
            if constexpr (FMB > 2) read_tok<2>(tok, st0, lane);
            if constexpr (FMB > 3) read_tok<3>(tok, st0, lane);
            static_assert(FMB <= 4, "prologue reads");
        }
        if (wave < DW) k_loop<true>(c, kt_begin, kt_end);
        else k_loop<false>(c, kt_begin, kt_end);
        // token loads of K-tiles past the end are still in flight: they must have landed before the
        // LDS is reused for the output tile or handed back
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (gridDim.y == 1) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the look-ahead fragment reads
            __syncthreads();
            Store::epilogue_lds(p, acc, m0, n0, 0, wave, lane, wave, lds);
        } else {
            Store::store_partials(p, acc, m0, n0, 0, wave, lane, split);
        }
    }
};

template <int TM, int TN, bool ROWMAJOR, bool NT>
__global__ void __launch_bounds__(512)
e4m3_bypass_kernel(LargeParams p) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
    typedef E4m3BypassKernel<TM, TN, ROWMAJOR, NT> Kern;
    Kern::run(p, lds_raw, (typename Kern::lds_byte *)lds_raw);
}

struct LargeConfig { int tm, tn, split, deep; double cost; int height; };     // height of the token tiles: tm or less (see cuts_tiles)

static const int kSplits[] = {1, 2, 3, 4, 6, 8};

// split-K cost: the reduction kernel's launch plus its traffic
static double split_cost(int64_t M, int64_t N, int slices, double launch_us, double bytes_per_us) {
    return launch_us + 8.0 * (double)M * (double)N * slices / bytes_per_us;
}

// At most 64 tokens: one 64 x 128 tile shape per weight kind and only the split to choose.  Such a
// launch is bound by the weight stream, whose rate depends on how many workgroups pull on it.
// Constants from timings of the four splits on six layer shapes at M = 64, packed planes.  Row-major planes
// share them, so that both storage orders launch alike and give the same bits, though by pairs of K-tiles
// (BypassKernel::PAIR) they hold one workgroup per CU: over 72 layer shapes at 20 ... 64 tokens the choice is
// 1.7 % (packed) and 2.3 % (row-major) behind the best split on average, 25 and 36 % at worst.
struct Tile64Cost {
    double tk, tfix;        // microseconds per K-tile and per workgroup
    int slots;              // workgroups the chip holds at a time
    double rate, rate512;   // bytes per microsecond of the weight stream (from 512 workgroups on)
    double few;             // exponent of the rate's fall below 256 workgroups
};
static const Tile64Cost kTile64Cost[3] = {
    {0.7, 0.4, 512, 4.5e6, 5.5e6, 0.5},       // plain FP16 (LDS kernel, three workgroups per CU)
    {0.466, 0.4, 512, 5.25e6, 5.5e6, 0.5},    // NestedFP16 (register path; packed planes: two per CU)
    {0.35, 0.4, 256, 5.5e6, 5.5e6, 0.3},      // E4M3 (register path, one per CU)
};
static LargeConfig choose_tile64(int cls, int64_t M, int64_t N, int64_t K, int max_split = 8) {
    const int kt = (int)(((cls == 2 ? K : 2 * K) + 127) / 128);
    const Tuning &t = tuning();
    const Tile64Cost &tc = kTile64Cost[cls];
    LargeConfig c;
    c.tm = 64;  c.tn = 128;  c.split = 1;  c.deep = 0;  c.height = 64;
    const int64_t tiles = ((M + 63) / 64) * ((N + 127) / 128);
    double best = 1e30;
    // A split stays inside the scratch of the entry point without a workspace wherever the problem does: the
    // streaming kernel, which may run the same layer, never needs more.  It bars splits of very wide layers only, which
    // fill the chip without: (57344, 8192) in FP16 mode at 64 tokens 199 us in the four slices the model
    // would take, 159 unsplit.  (Plain FP16 weights have no such entry point.)
    const bool bounded = cls != 0 && static_scratch_holds(1, M, N, K, cls == 2, partial_ld(N));
    for (int split : {1, 2, 3, 4, 6, 8}) {
        if (t.large_split > 0) split = (int)(t.large_split < kt ? t.large_split : kt);
        else if (split > 1 && (split > kt / 4 || split > max_split)) break;
        else if (bounded && !static_scratch_holds(split, M, N, K, cls == 2, partial_ld(N))) break;
        const int per = (kt + split - 1) / split;
        const int slices = (kt + per - 1) / per;
        const int64_t wgs = tiles * slices;
        const int64_t rounds = (wgs + tc.slots - 1) / tc.slots;
        double time = (double)rounds * (tc.tfix + per * tc.tk);
        double floor_t = (double)N * (double)kt * 128.0 / (wgs < 512 ? tc.rate : tc.rate512);
        if (wgs < 256) floor_t *= std::pow(256.0 / (double)wgs, tc.few);
        // the weight stream is shared per CU: workgroups beyond one per CU that do not make a whole
        // further round leave most CUs waiting for a few (measured: 320 workgroups take 1.3-1.5 times
        // as long as 240 with the same bytes)
        if (wgs > 256) floor_t *= (double)(((wgs + 255) / 256) * 256) / (double)wgs;
        if (time < floor_t) time = floor_t;
        if (slices > 1) time += split_cost(M, N, slices, 4.56, 4.24e6);
        if (time < best) { best = time;  c.split = split; }
        if (t.large_split > 0) break;
    }
    c.cost = best;
    // (a split whose scratch the padding of the rows has pushed past the fixed one: the best smaller split)
    if (t.large_split <= 0 && !padded_split_fits(c.split, M, N, K, cls == 2)) return choose_tile64(cls, M, N, K, c.split - 1);
    return c;
}

Tile64Plan tile64_plan(int kind, int64_t M, int64_t N, int64_t K) {
    static thread_local PlanCache<Tile64Plan> cache;
    return cache.get(kind_class(kind), M, N, K, [&] {
        const LargeConfig c = choose_tile64(kind_class(kind), M, N, K);
        return Tile64Plan{c.cost, c.split};
    });
}

// Token tiles of 256 exist cut down to 160, 192 and 224 tokens as well, all of a launch alike: register-path tiles and the
// 256 x 256 tiles of plain FP16 and E4M3.  The sums are the same at every height.
static bool cuts_tiles(int cls, int tn) { return cls == 1 || tn == 256; }
// Up to 256 tokens, and for timed launch shapes: the height that the batch needs, as many tiles as of 256 without the
// rows that only padding would fill.  777 tokens are four tiles of 224 instead of three of 256 and one of 9.  (28672, 4096),
// FP16 mode: 150 tokens 83.6 -> 66.9 us (row-major planes), 300 tokens 120 -> 96 us; FP8 mode gains 1-8 %.
static int token_tile(int cls, int tm, int tn, int64_t M) {
    if (tm != 256 || !cuts_tiles(cls, tn)) return tm;
    const int64_t tiles = (M + 255) / 256;
    const int h = (int)(((M + tiles - 1) / tiles + 31) / 32 * 32);
    return h < 160 ? 160 : h;
}
// the knob large_height instead, where there are such tiles
static int knob_height(int cls, int tm, int tn) {
    const int64_t want = tuning().large_height;
    return tm == 256 && cuts_tiles(cls, tn) && want >= 160 && want <= 256 && want % 32 == 0 ? (int)want : 0;
}

// Launch shapes that were timed faster than the cost model's choice, for the layer shapes of the
// models the paper evaluates (Sec. 5.1).  An entry tuned at M tokens serves the batches of more than
// 3 M / 4 (M / 2 up to 64 tokens) and at most M tokens that give the same number of token tiles.
// An entry holds no height of the token tiles: up to 256 tokens that is token_tile's, with the tile pinned for a timing as
// in the launch it stands for; above, the model would choose it, and the entry would be launched at another one than it was timed at.
struct TunedTile { int cls, N, K, M, tm, tn, split, deep; };
static constexpr TunedTile kTunedTiles[] = {
#include "tuned_tiles.inc"
    {-1, 0, 0, 0, 0, 0, 0, 0},
};
static constexpr bool tuned_up_to(int tokens) {
    for (const TunedTile &e : kTunedTiles)
        if (e.M > tokens) return false;
    return true;
}
static_assert(tuned_up_to(256), "timed launch shapes of more than 256 tokens need their height");

static bool tuned_large(int cls, int64_t M, int64_t N, int64_t K, LargeConfig &c) {
    for (const TunedTile &e : kTunedTiles) {
        if (e.cls != cls || e.N != N || e.K != K) continue;
        // (batches of up to 64 tokens are one 64-token tile whatever their size; above, a shape timed
        // at M tokens is trusted down to three quarters of M)
        if (M > e.M || (e.M <= 64 ? 2 * M <= e.M : 4 * M <= 3 * e.M)) continue;
        if ((M + e.tm - 1) / e.tm != (e.M + e.tm - 1) / e.tm) continue;
        c.tm = e.tm;  c.tn = e.tn;  c.split = e.split;  c.deep = e.deep;  c.height = token_tile(cls, e.tm, e.tn, M);
        return true;
    }
    return false;
}

// 65 ... 256 tokens of the two classes whose tiles of 256 tokens are cut down: every tile shape, the 64-token tiles
// included, priced by what was found to add up -- the rounds of workgroups, the weights, what all workgroups take in
// from L2 (weights and tokens) and what the busiest CU does.  Taken from timings of every shape and split (and both
// pipeline depths of E4M3, of which the deeper one is all that is left).  On the 82 000 launches that fit_costs.py times for them (weights
// cold, 70 layers of 0.8 to 500 Mi weights, twelve batch sizes, both storage orders) the choice is 2.2 % (FP16 mode) and 2.0 % (FP8
// mode) behind the fastest launch on average, 12-13 % at the 95th percentile; the model below, which knows neither the 64-token
// tiles nor the newer kernels, was 7-10 % behind.  Constants fitted to these timings are at 1.7 and 1.6 %, but take 40 to 90
// launches that lose more than 6 %; one launch timed twice differs by up to as much.
struct ShortShape { int tm, tn, deep; double tk, tfix, tk160, tfix160; };      // microseconds per K-tile and per workgroup; at a height of 160
struct ShortCost {
    ShortShape shape[5];
    double pair128, pair64;             // workgroups of a CU that run together
    double base, w_rate, l2_rate, cu_rate, split, split_rate;
};
static const ShortCost kShortCost[2] = {
    // FP16 operands through registers
    {{{256, 256, 0, 0.725, 6.05, 0.556, 3.47}, {256, 128, 0, 0.421, 2.63, 0.314, 1.28}, {128, 256, 0, 0.500, 2.61, 0, 0},
      {128, 128, 0, 0.2785, 0.83, 0, 0}, {64, 128, 0, 0.271, 0.51, 0, 0}}, 1.045, 1.045, 3.0, 15.2e6, 219e6, 167e3, 3.45, 5.28e6},
    // E4M3
    {{{256, 256, 0, 0.6255, 3.16, 0.378, 3.16}, {256, 128, 1, 0.319, 2.41, 0.319, 2.41}, {128, 256, 1, 0.334, 2.71, 0, 0},
      {128, 128, 1, 0.2136, 1.73, 0, 0}, {64, 128, 0, 0.183, 1.54, 0, 0}}, 1.0, 1.10, 2.0, 10.4e6, 1e15, 144e3, 3.28, 4.68e6},
};
// Splits whose partial sums outgrow the fixed scratch of nestedfp_gemm_static are left to FP16 mode, where they are priced 4 %
// cheaper than what fits: (17616, 5872) at 256 tokens in three slices of 18 MB 81 us (packed) and 93 (row-major), unsplit 103 and 111.
// (At 1-3 % they gain and lose by 10 %; in FP8 mode (8192, 28672) would gain 5-13 %, (5120, 32768) lose 12-21 %.)  That entry
// point takes what fits (bounded).
// E4M3 weights on 64-token tiles: the weight tiles past a multiple of eight (see tile_of_block) are fetched by each token tile on
// another XCD, from memory once the plane is larger than the L2s: with three and four token tiles such launches take 10-30 % longer than
// priced ((5840, 5840) at 144 tokens 29 us against 20.6 in two slices of 128 x 128), the others what they are priced at.
static LargeConfig choose_short(int cls, int64_t M, int64_t N, int64_t K, bool bounded) {
    const bool fp8 = cls == 2;
    const ShortCost &m = kShortCost[fp8 ? 1 : 0];
    const Tuning &t = tuning();
    const int kt = (int)(((fp8 ? K : 2 * K) + 127) / 128);
    const bool limited = static_scratch_holds(1, M, N, K, fp8, partial_ld(N));
    const int want_m = (t.large_bm == 128 || t.large_bm == 256) ? (int)t.large_bm : 0;
    const int want_n = (t.large_bn == 128 || t.large_bn == 256) ? (int)t.large_bn : want_m;
    LargeConfig c;
    c.tm = 128;  c.tn = 128;  c.split = 1;  c.deep = 0;  c.height = 128;
    double best = 1e30;
    for (const ShortShape &e : m.shape) {
        if (want_m && want_m != e.tm) continue;
        if (want_n && want_n != e.tn) continue;
        const int height = token_tile(cls, e.tm, e.tn, M);
        const int64_t tiles = ((M + e.tm - 1) / e.tm) * ((N + e.tn - 1) / e.tn);
        double tk = e.tk, tfix = e.tfix;
        if (e.tm == 256) {
            const double f = (height - 160) / 96.0;
            tk = e.tk160 + f * (e.tk - e.tk160);
            tfix = e.tfix160 + f * (e.tfix - e.tfix160);
        }
        for (int split : kSplits) {
            if (t.large_split > 0) split = (int)(t.large_split < kt ? t.large_split : kt);
            else if (split > 1 && split > kt / 4) break;
            const bool fits = t.large_split > 0 || !limited || static_scratch_holds(split, M, N, K, fp8, partial_ld(N));
            if (!fits && (fp8 || bounded || !padded_split_fits(split, M, N, K, fp8))) break;
            const int per = (kt + split - 1) / split;
            const int slices = (kt + per - 1) / per;
            const double wgs = (double)(tiles * slices), rounds = (double)((tiles * slices + 255) / 256);
            double time = rounds * (tfix + per * tk);
            if (rounds > 1 && e.tn == 128 && e.tm <= 128) time /= e.tm == 64 ? m.pair64 : m.pair128;
            time += m.base + (double)N * (double)K * (fp8 ? 1.0 : 2.0) / m.w_rate + wgs * per * (height + e.tn) * 128.0 / m.l2_rate +
                    rounds * per * (double)(std::min<int64_t>(height, M) + e.tn) * 128.0 / m.cu_rate;
            if (slices > 1) time += split_cost(M, N, slices, m.split, m.split_rate);
            if (!fits) time /= 0.96;
            if (fp8 && e.tm == 64 && M > 128 && (((N + 127) / 128) & 7) != 0 && N * K >= ((int64_t)24 << 20)) time *= 1.1;
            if (time < best) { best = time;  c.tm = e.tm;  c.tn = e.tn;  c.split = split;  c.deep = e.deep;  c.height = height; }
            if (t.large_split > 0) break;
        }
    }
    c.cost = best;
    return c;
}

// More than 256 tokens: tile shape, height of the token tiles and K split by the rounds of
// workgroups over 256 CUs, each a fixed time and a time per K-tile, the operands that all workgroups take in from L2,
// and what a split costs.  What is won over tiles of 256 tokens is the last round: (5888, 5888) at 1645 tokens is 161 tiles of
// 256 or 253 of 160, (6144, 4096) at 2048 tokens 192 or 240 of 224.  The constants were fitted to 112 000 timings of every shape,
// height and split worth one on 150 layers of 1 to 300 Mi weights at 272 to 8192 tokens, both storage orders, and to 40 000 more
// of FP8 mode with padded rows of codes (fit_costs.py time-tall and fit-tall take such timings and fit them).  Long K loops of the
// smaller tiles take more than their share (tk2): E4M3 on 128 x 128 tiles 13 % more at 100 K-tiles; (4064, 12208) at 589 tokens
// 73 us so, 60 in slices.  On the layers of the fit, and some left out of it, the choice was 0.5 to 0.6 % behind the fastest launch on
// average and 3.3 to 4.4 % at the 95th percentile; timed again on 159 layers, half of them drawn at random (114 000 timings of
// 4560 problems), 1.0 % (FP16 mode), 0.8 % (E4M3) and 1.1 % (plain FP16), and 6 to 9 %.  The model before it, which knew no
// heights, is 3.9, 4.3 and 4.5 % behind there, 16 to 19 %, but ahead by more than 3 % on 3 to 6 % of the problems, mostly small
// ones.  Constants fitted to these timings, with a term for rows that start inside lines, won 0.0 to 0.2 % on 855 further layers and slowed
// down as many calls as they sped up: not taken.
// Tiles of 128 tokens that all run at once, unsplit, read the same 128 bytes of K at the same time, and wait for memory
// together; a last token tile of few rows, which has half as much to load, runs ahead of the others and fetches their weights.
// Plain (2560, 2560) takes 28.5 us at 504 tokens, 28.9 at 767, but 21.5 at 649 and 776; in three and two slices, which start at
// other columns, 20.2 and 24.3.  Hence their price (lone, lone256; 2/5 is where the residuals of the prices part).  Timed with
// and without, weights cold, on 5622 problems drawn at 257 to 8192 tokens: behind the fastest launch 0.59 instead of 0.72 %
// (FP16 mode), 0.44 and 0.51 % (E4M3), 0.78 and 1.20 % (plain FP16), at the 95th percentile 4.0 and 4.8, 3.1 and 3.3, 5.4 and
// 8.0 %; slower by more than 3 % than the model without heights on 1.7 instead of 2.6, 0.9 and 1.3, 3.3 and 5.7 % of them.  The
// 140 problems whose launch it changes take 0.94 of the time; 22 of them are slower by 3 to 18 %, 90 faster by 3 to 22 %.
// That model still serves plain FP16 weights at 65 to 256 tokens, with the weights' one pass over the memory bus as a floor.  Launches
// that the floor prices alike are taken in the table's order, the larger tile first: (16142, 8128) at 125 tokens 80.7 us on 256 x 128
// tiles, 96.0 on 128 x 128 ones, and 12 to 25 % on 26 more of 65 to 128 tokens.
struct TallShape { int tm, tn, deep; double tk, tfix, tk160, tfix160, tk2; };       // as ShortShape; tk2: per K-tile squared
struct TallCost {
    int shapes;
    TallShape shape[7];
    double pair;                        // 128 x 128 workgroups of a CU that run together, from the second round on
    double l2_rate, split, split_rate;  // (no l2_rate: operands from L2 are not priced)
    double odd;                         // register path, rows on lines: slices of an odd number of K-tiles (see rows_through_lds)
    double lone, lone256;               // unsplit on 128 x 128 and 128 x 256 tiles, at most one workgroup per CU, the last token tile more than 2/5 full
    double floor_rate, floor_rate512;   // of the memory bus, slower while the chip is not full (from 512 workgroups on)
    bool both_depths;                   // every tile below 256 x 256 is priced in both pipelines, not 128 x 128 alone
};
static const TallCost kTallCost[4] = {
    // plain FP16 of up to 256 tokens
    {7, {{256, 256, 0, 1.353, 0, 1.353, 0, 0}, {256, 128, 0, 1.053, 0.07, 0, 0, 0}, {256, 128, 1, 0.863, 1.56, 0, 0, 0}, {128, 256, 0, 1.098, 0, 0, 0, 0},
         {128, 256, 1, 0.900, 1.71, 0, 0, 0}, {128, 128, 0, 0.848, 0, 0, 0, 0}, {128, 128, 1, 0.585, 2.50, 0, 0, 0}}, 1.58, 0, 3.18, 4.44e6, 1.0, 1.0, 1.0, 4.57e6, 4.44e6, true},
    // FP16 operands through registers
    {4, {{256, 256, 0, 1.11, 8.54, 0.773, 6.36, 0}, {256, 128, 0, 0.573, 6.03, 0.351, 5.53, 0.309e-3}, {128, 256, 0, 0.634, 6.39, 0, 0, 0.103e-3},
         {128, 128, 0, 0.285, 4.28, 0, 0, 0.466e-3}}, 1.0, 28.3e6, 2.98, 6.93e6, 1.05, 1.07, 1.0, 0, 0, false},
    // E4M3
    {5, {{256, 256, 0, 0.951, 9.83, 0.653, 7.57, 0}, {256, 128, 1, 0.445, 7.46, 0, 0, 0.502e-3}, {128, 256, 1, 0.598, 5.27, 0, 0, 0.026e-3},
         {128, 128, 0, 0.515, 4.75, 0, 0, 1.88e-3}, {128, 128, 1, 0.247, 5.41, 0, 0, 1.19e-3}}, 1.83, 50.5e6, 2.14, 5.55e6, 1.0, 1.09, 1.0, 0, 0, false},
    // plain FP16 above
    {5, {{256, 256, 0, 1.04, 7.72, 0.716, 5.68, 0}, {256, 128, 1, 0.466, 7.05, 0, 0, 0.286e-3}, {128, 256, 1, 0.578, 4.71, 0, 0, 0.168e-3},
         {128, 128, 0, 0.432, 4.88, 0, 0, 1.34e-3}, {128, 128, 1, 0.223, 4.69, 0, 0, 1.00e-3}}, 1.70, 34.3e6, 2.61, 6.13e6, 1.0, 1.12, 1.05, 0, 0, false},
};
// A split whose partial sums outgrow the fixed scratch of nestedfp_gemm_static is taken where it is priced 4 % below what fits,
// and by that entry point (bounded) nowhere: FP16 mode is 0.5 % behind the fastest launch so, 0.9 % if nothing beyond
// the scratch is taken.
static LargeConfig choose_tall(int cls, int64_t M, int64_t N, int64_t K, bool bounded) {
    const bool fp8 = cls == 2;
    const TallCost &m = kTallCost[cls == 0 && M > 256 ? 3 : cls];
    const Tuning &t = tuning();
    const int kt = (int)(((fp8 ? K : 2 * K) + 127) / 128);
    const bool limited = cls != 0 && static_scratch_holds(1, M, N, K, fp8, partial_ld(N));
    const int want_m = (t.large_bm == 128 || t.large_bm == 256) ? (int)t.large_bm : 0;
    const int want_n = (t.large_bn == 128 || t.large_bn == 256) ? (int)t.large_bn : want_m;
    LargeConfig c;
    c.tm = 128;  c.tn = 128;  c.split = 1;  c.deep = 0;  c.height = 128;
    double best = 1e30;
    for (int i = 0; i < m.shapes; ++i) {
        const TallShape &e = m.shape[i];
        if (want_m && want_m != e.tm) continue;
        if (want_n && want_n != e.tn) continue;
        int deep = e.deep;
        if (t.large_deep >= 0 && cls != 1 && !(e.tm == 256 && e.tn == 256)) {
            deep = t.large_deep > 0 ? 1 : 0;
            if (((e.tm == 128 && e.tn == 128) || m.both_depths) && deep != e.deep) continue;
        }
        const int pinned = knob_height(cls, e.tm, e.tn);
        const bool cut = e.tm == 256 && cuts_tiles(cls, e.tn);
        const int least = pinned ? pinned : (M <= 256 ? token_tile(cls, e.tm, e.tn, M) : (cut ? 160 : e.tm));
        const int most = pinned || M <= 256 ? least : e.tm;
        for (int height = least; height <= most; height += 32) {
            const double f = cut ? (height - 160) / 96.0 : 1.0;
            const double tk = e.tk160 + f * (e.tk - e.tk160), tfix = e.tfix160 + f * (e.tfix - e.tfix160);
            const int64_t tiles = ((M + height - 1) / height) * ((N + e.tn - 1) / e.tn);
            for (int split : kSplits) {
                if (t.large_split > 0) split = (int)(t.large_split < kt ? t.large_split : kt);
                else if (split > 1 && split > kt / 4) break;
                const bool fits = t.large_split > 0 || !limited || static_scratch_holds(split, M, N, K, fp8, partial_ld(N));
                if ((!fits && bounded) || (t.large_split <= 0 && !padded_split_fits(split, M, N, K, fp8))) break;
                const int per = (kt + split - 1) / split;                     // K-tiles per workgroup
                const int slices = (kt + per - 1) / per;
                const int64_t wgs = tiles * slices, rounds = (wgs + 255) / 256;
                double time = (double)rounds * (tfix + per * tk);
                if (rounds > 1 && e.tm == 128 && e.tn == 128 && !deep) time /= m.pair;
                time += (double)rounds * per * per * e.tk2;
                if (M <= 256 && cls == 0) {
                    double floor_t = (double)N * (double)K * 2.0 / (wgs < 512 ? m.floor_rate : m.floor_rate512);
                    if (wgs < 256) floor_t *= std::sqrt(256.0 / (double)wgs);
                    if (time < floor_t) time = floor_t;
                }
                if (m.l2_rate > 0) time += (double)wgs * per * (height + e.tn) * 128.0 / m.l2_rate;
                if (slices > 1) {
                    time += split_cost(M, N, slices, m.split, m.split_rate);
                    if ((per & 1) && (K & 127) == 0) time *= m.odd;
                } else if (e.tm == 128 && wgs <= 256 && 5 * ((M - 1) % 128 + 1) > 2 * 128) {
                    time *= e.tn == 128 ? m.lone : m.lone256;
                }
                if (!fits) time /= 0.96;
                if (time < best) { best = time;  c.tm = e.tm;  c.tn = e.tn;  c.split = split;  c.deep = deep;  c.height = height; }
                if (t.large_split > 0) break;
            }
        }
    }
    c.cost = best;
    return c;
}

static LargeConfig compute_large(int cls, int64_t M, int64_t N, int64_t K, bool bounded) {
    LargeConfig c;
    c.cost = 0.0;
    const Tuning &t = tuning();
    if (t.tuned_table != 0 && t.large_bm < 0 && t.large_bn < 0 && t.large_split <= 0 && t.large_deep < 0 && t.large_height < 0 &&
        tuned_large(cls, M, N, K, c))
        return c;
    if (t.large_bm == 64 || (M <= 64 && t.large_bm < 0 && t.large_bn < 0)) return choose_tile64(cls, M, N, K);
    const bool pinned = t.large_bm > 0 || t.large_bn > 0 || t.large_split > 0;
    if (M <= 256 && t.large_height < 0 && ((cls == 1 && t.large_deep <= 0) || (cls == 2 && t.large_deep < 0 && !pinned)))
        return choose_short(cls, M, N, K, bounded);
    return choose_tall(cls, M, N, K, bounded);
}

static LargeConfig choose_large(int kind, int64_t M, int64_t N, int64_t K, bool bounded) {
    static thread_local PlanCache<LargeConfig> cache;
    return cache.get(kind_class(kind) + (bounded ? 3 : 0), M, N, K, [&] { return compute_large(kind_class(kind), M, N, K, bounded); });
}

static size_t partial_bytes(const LargeConfig &c, int64_t M, int64_t N) {
    return c.split > 1 ? (size_t)c.split * (size_t)M * (size_t)partial_ld(N) * sizeof(float) : 0;
}
size_t large_gemm_partial_bytes(int kind, int64_t M, int64_t N, int64_t K) { return partial_bytes(choose_large(kind, M, N, K, false), M, N); }
size_t large_gemm_bounded_bytes(int kind, int64_t M, int64_t N, int64_t K) { return partial_bytes(choose_large(kind, M, N, K, true), M, N); }
int large_gemm_height(int kind, int64_t M, int64_t N, int64_t K) { return choose_large(kind, M, N, K, false).height; }

template <int KIND, int TM, int TN, int WAVES_M, int WAVES_N, int NST = 2, int NSTW = NST>
static void launch_large_t(const LargeParams &p, dim3 grid, hipStream_t stream) {
    auto kern = large_gemm_kernel<KIND, TM, TN, WAVES_M, WAVES_N, NST, NSTW>;
    constexpr int lds = LargeKernel<KIND, TM, TN, WAVES_M, WAVES_N, NST, NSTW>::LDS_BYTES;
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                            hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        attr_set.store(true, std::memory_order_release);
    }
    kern<<<grid, 64 * WAVES_M * WAVES_N, lds, stream>>>(p);
}

// Row-major planes that are read once (one token tile) and whose rows start on 128-byte lines are marked
// non-temporal like packed ones; where two pieces share a line it has to stay in L2.
static bool streams_rows(const LargeParams &p) {
    return p.tiles_m == 1 && (p.w_row_bytes & 127) == 0 && (reinterpret_cast<uintptr_t>(p.W0) & 127) == 0 &&
           (reinterpret_cast<uintptr_t>(p.W1) & 127) == 0;
}

// Packed weights on 64-token tiles are marked non-temporal with one token tile, which reads them once, and with several
// where all token tiles of a weight tile follow each other on one XCD (1.01-1.09 x faster so).  The weight tiles past a multiple of eight are
// read on several XCDs (see tile_of_block): on layers of 4 Mi weights and more, unmarked weights, which the memory-side cache keeps, are 2-13 %
// faster with two to four token tiles, and on FP16 layers of 64 Mi and more they are with any (6-8 %).  Timed both ways, weights cold,
// on 72 layers at 80, 128, 192 and 256 tokens in one to three slices.
static bool streams_tiles64(const LargeParams &p, bool fp8) {
    const int64_t weights = (int64_t)p.N * p.K, mi = (int64_t)1 << 20;
    return p.tiles_m == 1 || weights < 4 * mi || ((p.tiles_n & 7) == 0 && (fp8 || weights < 64 * mi));
}

template <int TM, int TN, int WK, bool DEEP = false, bool NT = false, bool PAIRS = false>
static void launch_bypass(const LargeParams &p, dim3 grid, hipStream_t stream) {
    auto kern = nested_bypass_kernel<TM, TN, WK, DEEP, NT, PAIRS>;
    constexpr int lds = BypassKernel<TM, TN, WK, DEEP, NT, PAIRS>::LDS_BYTES;
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        attr_set.store(true, std::memory_order_release);
    }
    kern<<<grid, 512, lds, stream>>>(p);
}

template <int TM, int TN, bool NT = false>
static void launch_rows(const LargeParams &p, dim3 grid, hipStream_t stream) {
    auto kern = nested_rows_kernel<TM, TN, NT>;
    constexpr int lds = RowsKernel<TM, TN, NT>::LDS_BYTES;
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        attr_set.store(true, std::memory_order_release);
    }
    kern<<<grid, 512, lds, stream>>>(p);
}

template <int TM, int TN, bool ROWMAJOR, bool NT = false>
static void launch_e4m3_bypass(const LargeParams &p, dim3 grid, hipStream_t stream) {
    if constexpr (!NT) {
        if (ROWMAJOR ? streams_rows(p) : streams_tiles64(p, true)) {
            launch_e4m3_bypass<TM, TN, ROWMAJOR, true>(p, grid, stream);
            return;
        }
    }
    auto kern = e4m3_bypass_kernel<TM, TN, ROWMAJOR, NT>;
    constexpr int lds = E4m3BypassKernel<TM, TN, ROWMAJOR, NT>::LDS_BYTES;
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        attr_set.store(true, std::memory_order_release);
    }
    kern<<<grid, 512, lds, stream>>>(p);
}

// weights through LDS: plain row-major FP16, E4M3 in either storage order
template <int KIND>
static void launch_large_k(const LargeParams &p, const LargeConfig &c, dim3 grid, hipStream_t stream) {
    if (c.height == 224) { launch_large_t<KIND, 224, 256, 2, 4, 2, 3>(p, grid, stream);  return; }
    if (c.height == 192) { launch_large_t<KIND, 192, 256, 2, 4, 2, 3>(p, grid, stream);  return; }
    if (c.height == 160) { launch_large_t<KIND, 160, 256, 2, 4, 3>(p, grid, stream);  return; }
    if (c.tm == 64) {
        if constexpr (KIND == kPlainF16) launch_large_t<KIND, 64, 128, 2, 4>(p, grid, stream);
        else launch_e4m3_bypass<64, 128, KIND == kE4M3Row>(p, grid, stream);
    } else if (c.tm == 256 && c.tn == 256) launch_large_t<KIND, 256, 256, 2, 4, 2, 3>(p, grid, stream);
    else if (c.tm == 256) {
        if (c.deep) launch_large_t<KIND, 256, 128, 4, 2, 3>(p, grid, stream);
        else launch_large_t<KIND, 256, 128, 4, 2>(p, grid, stream);
    } else if (c.tn == 256) {
        if (c.deep) launch_large_t<KIND, 128, 256, 2, 4, 3>(p, grid, stream);
        else launch_large_t<KIND, 128, 256, 2, 4>(p, grid, stream);
    } else {
        if (c.deep) launch_large_t<KIND, 128, 128, 2, 4, 4>(p, grid, stream);
        else launch_large_t<KIND, 128, 128, 2, 4>(p, grid, stream);
    }
}

// Row-major planes on the 64-token tiles and in the deeper pipeline of 128 tokens, 128 weight rows per tile: by pairs of K-tiles
// (see BypassKernel::PAIR; up to 45 % faster) where the longer look-ahead pays.  Timed both ways on 2760 launches (26 values
// of K from 512 to 17344, four N, twelve batch sizes, every split; tiles of 256 tokens among them): the rule was 0.4 % behind
// the faster way on average and at most 8 % behind unpaired loads (the rule "12 K-tiles per slice" 1.3 % and 23 %).
//  - Rows that start on lines: a dozen K-tiles per slice (64 tokens per tile 1.07-1.12 x at 12 K-tiles and 1.2 x at
//    24, 128 tokens 1.01 and 1.07); but not where the slices of a split have an odd number of K-tiles: every
//    second slice then starts in the middle of a line, its pieces take two lines each, and K-tile by K-tile
//    is 4-8 % faster.
//  - Rows that start inside lines: 14 K-tiles per slice, 6 Mi weights (smaller planes stay in the caches: K = 2064
//    at 100 tokens 0.97 x with N = 2048, 1.20 x with N = 5632), and longer rows the more token tiles read them
//    ((12288, 1600) at 128 tokens per tile: 1.11 x with one, 0.90 x with three).
bool rows_by_pairs(int tm, int64_t M, int64_t N, int64_t K, int64_t row_bytes, int split) {
    const int64_t kt = (K + 63) / 64, per = (kt + split - 1) / split, tiles_m = (M + tm - 1) / tm;
    const int64_t weights = N * K, mi = (int64_t)1 << 20;
    if ((row_bytes & 127) == 0) return per >= 12 && (per >= kt || (per & 1) == 0);
    if (per < 14) return false;
    if (tiles_m == 1) return weights >= (kt >= 24 ? 6 : 10) * mi;
    return weights >= 6 * mi && kt >= (tiles_m <= 4 ? 32 : 48);
}

// Row-major planes on the other tiles: through LDS by pairs of K-tiles (RowsKernel), or straight into registers in operand
// order, K-tile by K-tile.  Timed both ways by fit_costs.py on 17600 launches at 65 ... 256 tokens (70 layers, every tile shape
// and split, weights cold): the rule is 0.6 % behind the faster way on average, 5 % at the 95th percentile (everything
// straight into registers: 12 and 32 %); on 7200 launches of 300 ... 2048 tokens 0.3 and 2 % (8 %).
//  - Rows that start on lines: through LDS (1.01-1.06 x at less than a dozen K-tiles per slice, 1.15-1.24 x from three
//    dozen on), but on 128 x 128 tiles from a dozen K-tiles on (0.99 x on average below, 0.81 x at worst).
//  - Slices with an odd number of such K-tiles: every second one starts in the middle of a line, so that its pieces take
//    two lines each, and the last pair is half empty: a dozen K-tiles, but never on 256 x 256 tiles, whose two row tiles
//    per wave copy twice as much (1.02-1.07 x the time whatever the length; (5120, 14336) at 1024 tokens in slices of 75
//    K-tiles 170.7 us against 158.7).
//  - Rows that start inside lines, where pieces share lines but unpaired loads take whole halves if the row is a multiple
//    of 64 bytes: longer slices and rows, all the more where several token tiles read them from the caches.
bool rows_through_lds(int tm, int tn, int64_t M, int64_t K, int64_t row_bytes, int split) {
    const int64_t kt = (K + 63) / 64, per = (kt + split - 1) / split, tiles_m = (M + tm - 1) / tm;
    if ((row_bytes & 127) == 0) {
        if (per < kt && (per & 1)) return per >= 12 && !(tm == 256 && tn == 256);
        return per >= 12 || tm > 128 || tn > 128;
    }
    if ((row_bytes & 63) == 0) return per >= 20 && kt >= (tiles_m == 1 ? 24 : 48);
    return per >= 14 && kt >= (tiles_m == 1 ? 20 : 36);
}

template <int TM, bool DEEP>
static void launch_rows_by_pairs(const LargeParams &p, dim3 grid, hipStream_t stream) {
    const bool nt = streams_rows(p) && (TM == 64 || (int64_t)p.N * p.K >= ((int64_t)100 << 20));
    if (!rows_by_pairs(TM, p.M, p.N, p.K, p.w_row_bytes, (int)grid.y)) launch_bypass<TM, 128, kNestedF16Row, DEEP>(p, grid, stream);
    else if (nt) launch_bypass<TM, 128, kNestedF16Row, DEEP, true, true>(p, grid, stream);
    else launch_bypass<TM, 128, kNestedF16Row, DEEP, false, true>(p, grid, stream);
}

template <int TM, int TN>
static void launch_rows_tile(const LargeParams &p, dim3 grid, hipStream_t stream) {
    const int64_t knob = tuning().large_rows;
    const bool lds = knob >= 0 ? knob != 0 : rows_through_lds(TM > 128 ? 256 : 128, TN, p.M, p.K, p.w_row_bytes, (int)grid.y);
    if (!lds) {
        launch_bypass<TM, TN, kNestedF16Row>(p, grid, stream);
        return;
    }
    if constexpr (TM == 128 && TN == 128) {
        if (streams_rows(p) && (int64_t)p.N * p.K >= ((int64_t)100 << 20)) { launch_rows<TM, TN, true>(p, grid, stream);  return; }
    }
    launch_rows<TM, TN>(p, grid, stream);
}

// weights through registers: NestedFP16 in either storage order, packed FP16.  TM: the height of the token tiles
template <int WK, int TM>
static void launch_nested_tm(const LargeParams &p, const LargeConfig &c, dim3 grid, hipStream_t stream) {
    if constexpr (WK == kNestedF16Row) {
        if (c.tn == 128) launch_rows_tile<TM, 128>(p, grid, stream);
        else launch_rows_tile<TM, 256>(p, grid, stream);
    } else {
        if (c.tn == 128) launch_bypass<TM, 128, WK>(p, grid, stream);
        else launch_bypass<TM, 256, WK>(p, grid, stream);
    }
}

template <int WK>
static void launch_nested(const LargeParams &p, const LargeConfig &c, dim3 grid, hipStream_t stream) {
    if (c.height == 256) { launch_nested_tm<WK, 256>(p, c, grid, stream);  return; }
    if (c.height == 224) { launch_nested_tm<WK, 224>(p, c, grid, stream);  return; }
    if (c.height == 192) { launch_nested_tm<WK, 192>(p, c, grid, stream);  return; }
    if (c.height == 160) { launch_nested_tm<WK, 160>(p, c, grid, stream);  return; }
    if constexpr (WK == kNestedF16Row) {
        if (c.tm == 64) launch_rows_by_pairs<64, false>(p, grid, stream);
        else if (c.deep && c.tn == 128) launch_rows_by_pairs<128, true>(p, grid, stream);
        else if (c.deep) launch_bypass<128, 256, WK, true>(p, grid, stream);
        else launch_nested_tm<WK, 128>(p, c, grid, stream);
    } else if (c.tm == 64) {
        if (streams_tiles64(p, false)) launch_bypass<64, 128, WK, false, true>(p, grid, stream);
        else launch_bypass<64, 128, WK>(p, grid, stream);
    } else if (p.tiles_m == 1 && (int64_t)p.N * p.K >= ((int64_t)100 << 20)) {
        // one token tile over a large packed layer: weights marked non-temporal (see BypassKernel)
        if (c.tn == 256) {
            if (c.deep) launch_bypass<128, 256, WK, true, true>(p, grid, stream);
            else launch_bypass<128, 256, WK, false, true>(p, grid, stream);
        } else {
            if (c.deep) launch_bypass<128, 128, WK, true, true>(p, grid, stream);
            else launch_bypass<128, 128, WK, false, true>(p, grid, stream);
        }
    } else if (c.tn == 256) {
        if (c.deep) launch_bypass<128, 256, WK, true>(p, grid, stream);
        else launch_bypass<128, 256, WK>(p, grid, stream);
    } else {
        if (c.deep) launch_bypass<128, 128, WK, true>(p, grid, stream);
        else launch_bypass<128, 128, WK>(p, grid, stream);
    }
}

// The kernels address a tile with 32-bit byte offsets whose bit 31 marks a dead load, so 256 rows
// of any operand must stay below 2^31 bytes.
bool large_gemm_supports(int kind, int64_t K, int64_t ldx, int64_t ldw) {
    const int64_t x_row = kind_is_fp8(kind) ? ldx : 2 * ldx;
    const int64_t w_row = kind == kPlainF16 ? 2 * ldw : ((K + 63) / 64) * 64 * kind_elem_bytes(kind);
    const int64_t lim = (int64_t)1 << 31;
    return 256 * x_row + 4096 < lim && 256 * w_row + 4096 < lim;
}

int launch_large_gemm(int kind, const GemmArgs &a, hipStream_t stream) {
    if (!large_gemm_supports(kind, a.K, a.ldx, a.ldw)) return kErrShape;
    LargeConfig c = choose_large(kind, a.M, a.N, a.K, a.bounded);
    // the register-path kernels take the deeper pipeline only where it is asked for (knob) or was
    // timed faster (table), and only on the tiles of 128 tokens
    if (kind_class(kind) == 1) c.deep = (tuning().large_deep > 0 || (c.deep && tuning().large_deep != 0)) && c.tm == 128;
    // Workspaces are sized without the row stride of FP16 weights.  A matrix that spans 2 GiB or more comes here
    // with the scratch of the streaming kernel, which cannot address it: as many K slices as that holds.
    const size_t slice_bytes = (size_t)a.M * (size_t)partial_ld(a.N) * sizeof(float);
    const size_t room = a.partials != nullptr ? a.partial_bytes / slice_bytes : 0;
    if ((size_t)c.split > room) c.split = room > 1 ? (int)room : 1;
    LargeParams p;
    p.X = static_cast<const uint8_t *>(a.X);
    p.x_row_bytes = kind_is_fp8(kind) ? a.ldx : 2 * a.ldx;
    p.scales = a.scales;
    p.w_scale = a.w_scale;
    p.W0 = static_cast<const uint8_t *>(a.W0);
    p.W1 = static_cast<const uint8_t *>(a.W1);
    p.w_row_bytes = (kind == kPlainF16) ? 2 * a.ldw : a.K;        // row-major kinds only
    p.M = (int)a.M;  p.N = (int)a.N;  p.K = (int)a.K;
    p.k_bytes = kind_is_fp8(kind) ? (int)a.K : (int)(2 * a.K);
    p.kblocks = (int)((a.K + 63) / 64);
    p.Y = a.Y;  p.ldy = a.ldy;
    p.partials = a.partials;
    p.ldp = (int)partial_ld(a.N);
    p.tiles_m = (int)((a.M + c.height - 1) / c.height);
    p.tiles_n = (int)((a.N + c.tn - 1) / c.tn);
    p.ktiles_total = (p.k_bytes + 127) / 128;
    p.ktiles_per_split = (p.ktiles_total + c.split - 1) / c.split;
    c.split = (p.ktiles_total + p.ktiles_per_split - 1) / p.ktiles_per_split;   // no empty slices
    p.xcd_map = (tuning().large_xcd_map != 0 && p.tiles_m >= 2 && p.tiles_m < 8) ? 1 : 0;
    p.xcd_group = 0;
    if (tuning().large_xcd_map != 0 && p.tiles_m >= 8) {
        const int groups = (p.tiles_m + 5) / 6;
        p.xcd_group = (p.tiles_m + groups - 1) / groups;
    }
    p.rows_anywhere = ((a.N & 7) == 0 && (a.ldy & 7) == 0 && (reinterpret_cast<uintptr_t>(a.Y) & 15) == 0) ? 0 : 1;
    dim3 grid((unsigned)(p.tiles_m * p.tiles_n), (unsigned)c.split);
    switch (kind) {
        case kPlainF16: launch_large_k<kPlainF16>(p, c, grid, stream); break;
        case kNestedF16: launch_nested<kNestedF16>(p, c, grid, stream); break;
        case kNestedF16Row: launch_nested<kNestedF16Row>(p, c, grid, stream); break;
        case kPlainF16Packed: launch_nested<kPlainF16Packed>(p, c, grid, stream); break;
        case kE4M3: launch_large_k<kE4M3>(p, c, grid, stream); break;
        case kE4M3Row: launch_large_k<kE4M3Row>(p, c, grid, stream); break;
        default: return kErrArg;
    }
    if (hipGetLastError() != hipSuccess) return kErrHip;
    if (c.split > 1)
        return launch_splitk_reduce(a.partials, c.split, a.M, a.N, kind_is_fp8(kind) ? a.scales : nullptr,
                                    a.w_scale, a.Y, a.ldy, stream);
    return kOk;
}

}  // namespace nfp
