// Dequantize-and-contract kernel of the adapted layer for gfx950 (Alg. 1 qblora_forward: W_tilde = dequantize(...),
// x @ W_tilde, plus the adapter term; and dX of its backward, on the transposed weight), for calls that do not
// dequantize the weight beforehand: few tokens on wide layers, and the forward that allocates nothing.
//
//   C[M,N] = X1[M,K1] * Wq^T  +  X2[M,K2] * W2[N/div2, K2]^T     (forward: N = d_out, K1 = d_in; dX: the other way)
//
// Segment 1 reads the 4-bit codes and block scales of the frozen base weight from HBM, rebuilds
// bf16 weights (Eq. 1: c[code]*alpha (+beta), fp32 then round-to-nearest-even) straight into an
// LDS tile and feeds them to v_mfma_f32_16x16x32_bf16 with fp32 accumulation; the dequantized
// weight never exists in HBM.  Segment 2 is a plain bf16 K-extension: the adapter's rank-R product
// rides in the same accumulators as R extra contraction steps (X2 = s*U, W2 = B^T with output row n using row
// n/lambda2, i.e. repeat_interleave; dX: X2 = dU/lambda1, W2 = A with row k/lambda1).  k is accumulated in the order and
// by the instruction of dense.hip, so both give the same bits.
//
// Shape of the computation on a CU: one workgroup of 512 threads (8 wave64, two per SIMD) owns 256 tokens x 256 or 128
// features; a wave owns 128 x 64 or 64 x 64 of them (128 or 64 accumulator registers).  Two waves per SIMD matter: the
// dequantization arithmetic of one wave issues in the shadow of the other wave's MFMAs.  Both operand tiles live in LDS
// as [row][64 k] bf16 (128 bytes per row) with the 16-byte chunks of a row XOR-swizzled by (row >> 1) & 7, double
// buffered, one barrier per k-step.  Activation tiles (and both bf16 tiles of segment 2) go from global memory directly
// into LDS (global_load_lds, 16 bytes per lane; the swizzle is applied by choosing which global chunk a lane fetches).
// Codes and block parameters are fetched two or three k-steps ahead into registers and dequantized between the MFMAs of
// the step before they are needed, through a byte-indexed table in LDS that turns one byte of codes into two fp32
// code values.  The transposed form stages a patch of 4 or 2 stored rows x 8 columns per thread and packs it down the
// columns; its scales, one a row, are spread inside a quad of lanes.  It takes as long as the other.
//
// Bound: LDS.  A 64-wide step of the 256 x 256 tile reads 192 KB of fragments and 64 KB of table values and writes 64 KB,
// about 2600 cycles of LDS against 2048 of MFMAs; it takes 1.5 us with few workgroups and 1.85 us (power) with all CUs
// busy, the 256 x 128 tile 0.95 and 1.08.  No form may spill: with accumulators, fragments, table values and the codes
// in flight the wide tile needs nearly all 256 registers, and a version that kept the code row pointers, the
// K-extension's addresses and four scales a thread in them spilled inside its loop (8 x 8 blocks with offsets 217 us at
// 512 tokens, 4096 x 4096, where this one takes 61).  Hence 32-bit lane offsets from uniform bases, addresses made again
// where they are used, and with 8 x 8 blocks a thread that owns one column of one block: one scale, one offset.
//
// The weight tile is the MFMA A operand and the token tile the B operand, so a lane ends up with 4
// consecutive output features of one token and stores them as one 8-byte word.
#include <type_traits>

#include "common.h"

namespace qblora {

namespace {

constexpr int kThreads = 512;
constexpr int BM = 256, kBK = 64;
constexpr int kTileX = BM * 128;                            // a token tile: rows of 128 bytes
constexpr int kTableBytes = 256 * 128;                      // byte-indexed pair table, 16 replicas

__device__ __align__(16) const uint32_t g_zero_chunk[4] = {0u, 0u, 0u, 0u};

// Byte of a 16-byte chunk in a weight tile.  TR: its columns are written by threads 8 tile rows apart, which the row's low
// bits alone would send to two chunk positions; the number of the 16-row block spreads them over all eight.
template <bool TR>
__device__ __forceinline__ int swz_w(int row, int chunk) {
    return row * 128 + (((chunk ^ (row >> 1) ^ (TR ? row >> 4 : 0)) & 7) << 4);
}

// One wave-wide global -> LDS copy: lane i fetches 16 bytes and they land at lds_base + 16*i (M0
// carries the wave-uniform LDS byte address).  Written as assembly so that the compiler's wait-count
// bookkeeping does not tie later LDS accesses to these copies; every copy is completed by the
// explicit vmcnt(0) in front of the barrier that publishes the tile.
__device__ __forceinline__ void copy16_to_lds(const void* src, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 :: "s"(lds_base), "v"(src) : "memory");
}
__device__ __forceinline__ void copy16_to_lds(const void* uniform_base, uint32_t lane_offset, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_base), "v"(lane_offset), "s"(uniform_base) : "memory");
}

__device__ __forceinline__ uint32_t lds_address(const void* p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

// Codes and block parameters of one k-step held in registers: D dwords of 8 codes per thread.  The weight itself: all in
// one block -- consecutive dwords of a stored row, or, with 8 x 8 quantization blocks, the same 8 inputs of D adjacent
// rows.  Transposed: the same 8 columns of D adjacent stored rows; the scale is that of row (lane % D) of those, which
// the lanes of a quad share (they hold 32 consecutive columns), or with 8 x 8 blocks the one of all.
template <int D>
struct Staged {
    uint32_t cw[D];
    float sc, be;
};

// v of lane I of the caller's aligned group of D lanes (D = 2 or 4)
template <int D, int I>
__device__ __forceinline__ float group_broadcast(float v) {
    constexpr int quad = D == 4 ? I * 0x55 : I == 0 ? 0xA0 : 0xF5;        // quad_perm
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), quad, 0xf, 0xf, false));
}

// The lane, read again where it is used: a value that need not be kept in a register across the loop.
__device__ __forceinline__ int lane_id() {
    int l = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(l));
    return l;
}

typedef __attribute__((ext_vector_type(2))) float f32x2;

template <int N> using Int = std::integral_constant<int, N>;

// Waits until at most N of this wave's loads and copies are in flight and its LDS accesses are done, then the
// workgroup's barrier.  The builtin tells the compiler that its own loads up to there have arrived; the statement keeps
// every memory access on its side of the barrier.
template <int N>
__device__ __forceinline__ void publish(Int<N>) {
    static_assert(N >= 0 && N < 16, "one field of the wait");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0070 | N);
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// TR: the transposed weight (output features = stored columns, contraction over stored rows)
template <int BN, bool BETA, int BR, bool TR>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_qlinear(GemmDesc d) {
    constexpr int kTileW = BN * 128, D = BN / 64;    // bytes of a weight tile, code dwords per thread and step
    constexpr int MB = BN / 32;                      // 16-token blocks of a wave
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* const sW = smem + 2 * kTileX;                // 2 token tiles in front, then 2 weight tiles
    unsigned char* const sT = sW + 2 * kTileW;                  // pair table, see below

    // Every field of the descriptor the loop touches is copied into a local first: the copies in
    // the loop are assembly statements that clobber memory, and values must not be re-read around them.
    const int64_t M = d.M;
    const int N = d.N, d_in = d.d_in, K2 = d.K2, div2 = d.div2;
    const qblora_bf16* const X1 = d.X1; const int64_t ldx1 = d.ldx1;
    const qblora_bf16* const X2 = d.X2; const int64_t ldx2 = d.ldx2;
    const qblora_bf16* const W2 = d.W2; const int64_t ldw2 = d.ldw2;
    const float* const beta = d.beta;
    qblora_bf16* const C = reinterpret_cast<qblora_bf16*>(d.C);
    const int64_t ldc = d.ldc;
    const float out_scale = d.out_scale;

    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    // a wave owns 16*MB tokens x 64 features
    const int wm0 = BN == 256 ? (wave & 1) * 128 : (wave & 3) * 64, wn0 = BN == 256 ? (wave >> 1) * 64 : (wave >> 2) * 64;

    // ---- tile assignment: XCD-contiguous, grouped along tokens ---------------------------------
    const int tiles_m = (int)((M + BM - 1) / BM), tiles_n = (N + BN - 1) / BN;
    const int ntiles = tiles_m * tiles_n;
    int L;
    {
        const int xcd = blockIdx.x & 7, q = ntiles >> 3, rem = ntiles & 7;
        L = xcd * q + min(xcd, rem) + (blockIdx.x >> 3);
    }
    constexpr int GM = 4;
    const int in_group = GM * tiles_n;
    const int first_m = (L / in_group) * GM;
    const int gsize = min(tiles_m - first_m, GM);
    const int mt = first_m + (L % in_group) % gsize, nt = (L % in_group) / gsize;
    const int64_t m0 = (int64_t)mt * BM;
    const int n0 = nt * BN;

    const int steps1 = (TR ? d.d_out : d_in) / kBK, steps2 = (K2 + kBK - 1) / kBK;
    const int nsteps = steps1 + steps2;
    const int bpr = d_in / kBlock;                // blocks per stored weight row

    f32x4 acc[4][MB];                             // [16 features][16 tokens]
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < MB; ++b) acc[a][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // ---- direct global -> LDS copies -------------------------------------------------------------
    // Wave w fills rows 32w .. 32w+31 of a token tile (BN/8 rows of a weight tile) with copies of 8 rows each.  In
    // copy i, lane l lands on row 8i + (l>>3) of those, physical chunk l&7, which must hold logical chunk
    // (l&7) ^ (row>>1)&7 = (l&7) ^ (4(i&1) + (l>>4)).
    const int crow = lane >> 3;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem));
    // a tile of the K-extension: chunks at or beyond K2 are fetched from a zero constant instead
    auto copy_tile = [&](auto rows_per_wave, const qblora_bf16* src, int64_t ld, int64_t row_base, int64_t row_max,
                         int div, int k0, uint32_t tile_off, const bool weight) __attribute__((always_inline)) {
        const int l = lane_id();                     // row addresses are made again at every call, not held across the loop
#pragma unroll
        for (int i = 0; i < rows_per_wave.value / 8; ++i) {
            int64_t row = row_base + wave * rows_per_wave.value + i * 8 + (l >> 3);
            row = row > row_max ? row_max : row;
            if (div != 1) row = (int64_t)((uint32_t)row / (uint32_t)div);      // only weight rows (< 2^31) are divided
            const int high = TR && weight ? ((wave * rows_per_wave.value + i * 8) >> 4) & 7 : 0;    // see swz_w
            const int k = k0 + (((l & 7) ^ (4 * (i & 1) + (l >> 4)) ^ high) << 3);
            const qblora_bf16* p = k < K2 ? src + row * ld + k : reinterpret_cast<const qblora_bf16*>(g_zero_chunk);
            copy16_to_lds(p, lds0 + tile_off + (wave * rows_per_wave.value + i * 8) * 128);
        }
    };
    // Segment-1 activation tiles: per-lane byte offsets relative to the tile's first row are fixed for
    // the whole kernel, the uniform base walks along k.
    uint32_t xoff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int64_t lrow = wave * 32 + i * 8 + crow;
        if (m0 + lrow > M - 1) lrow = M - 1 - m0;
        xoff[i] = (uint32_t)(lrow * ldx1 * 2) + (((lane & 7) ^ (4 * (i & 1) + (lane >> 4))) << 4);
    }
    const qblora_bf16* const x1_tile = X1 + m0 * ldx1;
    auto issue_x1 = [&](int step) __attribute__((always_inline)) {
        const qblora_bf16* base = x1_tile + (int64_t)step * kBK;
        const uint32_t to = lds0 + (step & 1) * kTileX + wave * 32 * 128;
#pragma unroll
        for (int i = 0; i < 4; ++i) copy16_to_lds(base, xoff[i], to + i * 8 * 128);
    };
    auto issue_copies = [&](int step) __attribute__((always_inline)) {
        if (step < steps1) {
            issue_x1(step);
        } else {
            const int k0 = (step - steps1) * kBK, buf = step & 1;
            copy_tile(Int<32>{}, X2, ldx2, m0, M - 1, 1, k0, buf * kTileX, false);
            copy_tile(Int<BN / 8>{}, W2, ldw2, n0, N - 1, div2, k0, 2 * kTileX + buf * kTileW, true);
        }
    };

    // ---- codes / scales -> registers -------------------------------------------------------------
    // 64-blocks: a thread owns 1/(512/BN) of a stored row.  8 x 8 blocks: the dword t & 7 of D rows of one block row.
    // Transposed: 8 columns of D stored rows.  wrow / wchunk: its place in the tile, of the first of its columns if TR.
    constexpr int kPerRow = 512 / BN, kGroups = BN / 8;
    const int wrow = TR ? 8 * (t % kGroups) : BR == 8 ? D * (t >> 3) : t / kPerRow;
    const int wchunk = TR ? D * (t / kGroups) / 8 : BR == 8 ? (t & 7) : D * (t % kPerRow);
    // (uniform bases, which walk along k, and 32-bit lane offsets from the tile's first row or column; rows past N: any
    // valid ones, results never stored)
    const uint8_t* codes_at; int64_t codes_step = 32;
    const float *scales_at, *beta_at = nullptr;
    uint32_t codes_off, codes_row = (uint32_t)(d_in / 2), scales_off, blk_off;
    if constexpr (TR) {
        const int row = D * (t / kGroups), col = min(n0 + wrow, N - 8) - n0;
        codes_at = d.codes + n0 / 2; codes_step = 32 * (int64_t)d_in;
        codes_off = (uint32_t)row * codes_row + (uint32_t)(col / 2);
        blk_off = BR == 8 ? (uint32_t)(row >> 3) * (uint32_t)(d_in >> 3) + (uint32_t)(n0 + col) / 8u
                          : (uint32_t)(row + (t & (D - 1))) * (uint32_t)bpr + (uint32_t)(n0 + col) / kBlock;
        scales_off = blk_off;
        scales_at = d.scales;
        if constexpr (BETA) beta_at = beta;
    } else {
        const int lrow = min(n0 + wrow, N - (BR == 8 ? D : 1)) - n0;
        codes_off = (uint32_t)lrow * codes_row;
        if (d.codes_tiled) { codes_at = d.codes_tiled + tiled_run_offset(n0, 0, bpr); codes_step = 256 * 32; codes_row = 32; codes_off = (uint32_t)lrow * 32u; }
        else codes_at = d.codes + (int64_t)n0 * (d_in / 2);
        codes_off += (uint32_t)wchunk * 4u;
        const int64_t blk0 = BR == 8 ? (int64_t)(n0 >> 3) * (d_in >> 3) : (int64_t)n0 * bpr;
        blk_off = BR == 8 ? (uint32_t)(lrow >> 3) * (uint32_t)(d_in >> 3) + (uint32_t)wchunk : (uint32_t)lrow * (uint32_t)bpr;
        // 64-blocks: the scales come in tile order
        scales_at = BR == 8 ? d.scales + blk0 : d.scales_tiled + tiled_run_offset(n0, 0, bpr) / 32;
        scales_off = BR == 8 ? blk_off : (uint32_t)lrow;
        if constexpr (BETA) beta_at = beta + blk0;
    }
    const int64_t scales_step = TR ? d_in : BR == 8 ? 8 : 256, beta_step = TR ? d_in : BR == 8 ? 8 : 1;
    constexpr bool kRows = TR || BR == 8;                            // a dword of each of D stored rows
    constexpr int kLoads = (kRows ? D : 1) + 1 + (BETA ? 1 : 0);     // load instructions of a step
    typedef typename std::conditional<D == 4, u32x4_any, u32x2_any>::type Row;
    auto load_staged = [&](Staged<D>& s, int step) __attribute__((always_inline)) {
        const uint8_t* const p = codes_at + step * codes_step;
        if constexpr (kRows) {
#pragma unroll
            for (int i = 0; i < D; ++i) s.cw[i] = *reinterpret_cast<const u32_any*>(p + codes_row * i + codes_off);
        } else {
            const Row v = *reinterpret_cast<const Row*>(p + codes_off);
#pragma unroll
            for (int i = 0; i < D; ++i) s.cw[i] = v[i];
        }
        s.sc = (scales_at + step * scales_step)[scales_off];
        if constexpr (BETA) s.be = (beta_at + step * beta_step)[blk_off];
        asm volatile("" ::: "memory");               // the loads stay in front of what follows
    };

    // ---- dequantization of a staged k-step, in 4*D units of one byte of codes (two adjacent inputs) -----------------
    // The weight itself: unit u is byte u & 3 of dword u / 4, and four units fill a 16-byte chunk.  Transposed: byte u / D
    // of stored row u % D; the D rows of a byte are packed down its two columns.
    const uint32_t table_lane = lds_address(sT) + ((lane & 15) << 3);
    auto look_up = [&](const Staged<D>& s, int u) __attribute__((always_inline)) {
        const uint32_t w = s.cw[TR ? u % D : u / 4];
        const int i = TR ? u / D : u % 4;
        const uint32_t at = ((i == 0 ? (w << 7) : (w >> (8 * i - 7))) & 0x7f80u) | table_lane;
        return *reinterpret_cast<const __attribute__((address_space(3))) f32x2*>(at);
    };
    float rs[D], rb[D];                              // transposed 64-blocks: of the D rows of the tile in work
    auto spread = [&](const Staged<D>& s) __attribute__((always_inline)) {
        if constexpr (TR && BR == 1) {
            rs[0] = group_broadcast<D, 0>(s.sc); rs[1] = group_broadcast<D, 1>(s.sc);
            if constexpr (BETA) { rb[0] = group_broadcast<D, 0>(s.be); rb[1] = group_broadcast<D, 1>(s.be); }
            if constexpr (D == 4) {
                rs[2] = group_broadcast<D, 2>(s.sc); rs[3] = group_broadcast<D, 3>(s.sc);
                if constexpr (BETA) { rb[2] = group_broadcast<D, 2>(s.be); rb[3] = group_broadcast<D, 3>(s.be); }
            }
        }
    };
    auto scaled = [&](float c, float sc, float be) __attribute__((always_inline)) { return BETA ? __fmaf_rn(c, sc, be) : __fmul_rn(c, sc); };
    uint32_t store_at = TR ? (uint32_t)(swz_w<TR>(wrow, wchunk) + (D * (t / kGroups) % 8) * 2) : (uint32_t)swz_w<TR>(wrow, wchunk);
    uint32_t o[4];
    // lv: the values of units u & ~3 .. | 3
    auto finish = [&](const Staged<D>& s, int u, const f32x2 (&lv)[4], unsigned char* tile) __attribute__((always_inline)) {
        if constexpr (!TR) {
            const f32x2 c = lv[u & 3];
            o[u & 3] = pack_bf16(scaled(c[0], s.sc, s.be), scaled(c[1], s.sc, s.be));
            if ((u & 3) != 3) return;
            // swz(wrow, wchunk + p), or swz(wrow + p, wchunk) with 8 x 8 blocks: wchunk and wrow are multiples of D
            const int p = u >> 2;
            const uint32_t at = BR == 8 ? (store_at ^ (uint32_t)((p >> 1) << 4)) + p * 128 : store_at ^ (uint32_t)(p << 4);
            *reinterpret_cast<uint4*>(tile + at) = make_uint4(o[0], o[1], o[2], o[3]);
        } else {
            const int i = u % D, p = u / D;
            if ((i & 1) == 0) return;
            const f32x2 c0 = lv[(u - 1) & 3], c1 = lv[u & 3];        // stored rows i - 1 and i
            const float s0 = BR == 8 ? s.sc : rs[(i - 1) % D], s1 = BR == 8 ? s.sc : rs[i];
            const float b0 = !BETA ? 0.0f : BR == 8 ? s.be : rb[(i - 1) % D], b1 = !BETA ? 0.0f : BR == 8 ? s.be : rb[i];
            o[i >> 1] = pack_bf16(scaled(c0[0], s0, b0), scaled(c1[0], s1, b1));            // column 2p
            o[2 + (i >> 1)] = pack_bf16(scaled(c0[1], s0, b0), scaled(c1[1], s1, b1));      // column 2p + 1
            if (i != D - 1) return;
            unsigned char* const at = tile + (store_at ^ (uint32_t)(p << 4)) + p * 256;     // two tile rows share a swizzle
            if constexpr (D == 2) {
                *reinterpret_cast<uint32_t*>(at) = o[0];
                *reinterpret_cast<uint32_t*>(at + 128) = o[2];
            } else {
                *reinterpret_cast<uint2*>(at) = make_uint2(o[0], o[1]);
                *reinterpret_cast<uint2*>(at + 128) = make_uint2(o[2], o[3]);
            }
        }
    };

    // ---- fragments ----------------------------------------------------------------------------------
    // 16-row block b, slice ks of 32 k: row base + 16b + r, chunk 4ks + g sits at (base + r)*128 + 2048b +
    // 16*[(g ^ r>>1) & 7 ^ 4ks] -- one per-lane value XOR a constant plus an immediate;
    // the empty asm in a step keeps the variants from being hoisted and held in registers.
    const int r = lane & 15, g = lane >> 4;
    // (the transposed weight's tile: XOR the number of the 16-row block as well)
    uint32_t frag_w = 2 * kTileX + (uint32_t)((wn0 + r) * 128 + (((g ^ (r >> 1)) ^ (TR ? (wn0 >> 4) & 7 : 0)) << 4));
    uint32_t frag_x = (uint32_t)((wm0 + r) * 128 + ((g ^ (r >> 1)) << 4));
    auto read_w = [&](int buf, int ks, bf16x8 (&f)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < 4; ++a)
            f[a] = *reinterpret_cast<const bf16x8*>(smem + ((frag_w ^ (uint32_t)((ks << 6) ^ (TR ? a << 4 : 0))) + buf * kTileW) + a * 2048);
    };
    auto read_x = [&](int buf, int ks, int half, bf16x8 (&f)[4]) __attribute__((always_inline)) {
        const unsigned char* const p = smem + ((frag_x ^ (uint32_t)(ks << 6)) + buf * kTileX) + half * 8192;
#pragma unroll
        for (int b = 0; b < 4; ++b) f[b] = *reinterpret_cast<const bf16x8*>(p + b * 2048);
    };
    auto mfma = [&](const bf16x8& w, const bf16x8& x, f32x4& c) __attribute__((always_inline)) {
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, x, c, 0, 0, 0);
    };

    // ---- one k-step ----------------------------------------------------------------------------------
    // Buffer s & 1 of both tiles holds step s when it starts, and the copies of step s+1's tokens are in flight.  Its
    // barrier publishes tile s+1 and frees the buffers of step s.  A wave issues in order, so the dequantization is
    // written between the MFMAs in whose shadow it runs, and fenced there.
    // kMode 1: steps s+1 and s+2 are quantized, no conditions (codes are fetched ahead from a clamped step); 0: the last
    // quantized steps; 2: the K-extension, nothing to dequantize.
    constexpr int kSets = BN == 256 ? 2 : 4;
    Staged<D> st[kSets];                             // by step % kSets
    bf16x8 wf[BN == 256 ? 1 : 2][4], xf[BN == 256 ? 1 : 2][4];
    f32x2 lv[2][4];                                  // table values of two chunks
    auto step = [&](auto mode, auto phase, int s) __attribute__((always_inline)) {
        constexpr int kMode = mode.value, P = phase.value;
        const int cur = s & 1, nxt = cur ^ 1;
        const bool dq = kMode == 1 || (kMode == 0 && s + 1 < steps1), look = kMode == 1 || (kMode == 0 && s + 2 < steps1);
        const bool more = kMode == 1 || s + 1 < nsteps;
        unsigned char* const w_next = sW + nxt * kTileW;
        asm volatile("" : "+v"(frag_w), "+v"(frag_x), "+v"(store_at));
        if constexpr (BN == 128) {
            // First slice: its MFMAs, weight tile s+1 scaled and stored (looked up in the step before), the second slice's
            // fragments read.  Second slice: 6 MFMAs, the barrier, then the other 10 beside the reads of tile s+1's
            // first fragments, the copies of step s+2 and its lookups.  Codes are fetched three steps ahead; those of
            // this step stay in flight across the barrier.
            if (kMode == 1 || (kMode == 0 && s + 3 < steps1)) load_staged(st[(P + 3) & 3], min(s + 3, steps1 - 1));
            read_w(cur, 1, wf[1]);
            read_x(cur, 1, 0, xf[1]);
            if (dq) spread(st[(P + 1) & 3]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                mfma(wf[0][i >> 2], xf[0][i & 3], acc[i >> 2][i & 3]);
                if (i < 8 && dq) finish(st[(P + 1) & 3], i, lv[i >> 2], w_next);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int i = 0; i < 6; ++i) mfma(wf[1][i >> 2], xf[1][i & 3], acc[i >> 2][i & 3]);
            if constexpr (kMode == 1) publish(Int<kLoads>{}); else publish(Int<0>{});
            if (more) { read_w(nxt, 0, wf[0]); read_x(nxt, 0, 0, xf[0]); }
            if (kMode == 1) issue_x1(s + 2);
            else if (s + 2 < nsteps) issue_copies(s + 2);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 6; i < 16; ++i) {
                mfma(wf[1][i >> 2], xf[1][i & 3], acc[i >> 2][i & 3]);
                const int u = i - 6;
                if (u < 8 && look) lv[u >> 2][u & 3] = look_up(st[(P + 2) & 3], u);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            // Four quarters of 16 MFMAs: a 32-wide slice of k, half of the wave's tokens.  There are no registers for a
            // second set of fragments: the MFMAs of a quarter run along the antidiagonals of [feature block][token
            // block], so that every fragment is replaced by the next quarter's behind its last use and has five or more
            // MFMAs to arrive.  The next weight tile is scaled and stored over the first three quarters, its table values
            // read four units ahead; the barrier stands behind 6 MFMAs of the last quarter, in front of the first read
            // of the next tiles.  Codes are fetched two steps ahead.
            if (kMode == 1 || (kMode == 0 && s + 2 < steps1)) load_staged(st[P & 1], min(s + 2, steps1 - 1));
            if (dq) spread(st[(P + 1) & 1]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t slice = q == 1 || q == 2 ? 64 : 0;          // of quarter q + 1
                const unsigned char* const xs = smem + ((frag_x ^ slice) + (q < 3 ? cur : nxt) * kTileX) + ((q + 1) & 1) * 8192;
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0, n = 0; j < 7; ++j) {
#pragma unroll
                    for (int a = 0; a < 4; ++a) {
                        const int b = j - a;
                        if (b < 0 || b > 3) continue;
                        mfma(wf[0][a], xf[0][b], acc[a][(4 * (q & 1) + b) % MB]);
                        const int m = 16 * q + n, u = m / 3;
                        if (q < 3 && m % 3 == 0 && dq) {
                            finish(st[(P + 1) & 1], u, lv[(u >> 2) & 1], w_next);
                            if (u < 12) lv[((u >> 2) + 1) & 1][u & 3] = look_up(st[(P + 1) & 1], u + 4);
                        }
                        if (q == 3 && n == 5) {
                            publish(Int<0>{});
                            if (kMode == 1) issue_x1(s + 2);
                            else if (s + 2 < nsteps) issue_copies(s + 2);
                        }
                        if (q == 3 && n > 5 && n % 2 == 1 && n < 15 && look) lv[0][(n - 7) / 2] = look_up(st[P & 1], (n - 7) / 2);
                        if (b == 3 && (q & 1) && (q < 3 || more)) 
                            wf[0][a] = *reinterpret_cast<const bf16x8*>(
                                smem + ((frag_w ^ slice ^ (uint32_t)(TR ? a << 4 : 0)) + (q < 3 ? cur : nxt) * kTileW) + a * 2048);
                        if (a == 3 && (q < 3 || more)) xf[0][b] = *reinterpret_cast<const bf16x8*>(xs + b * 2048);
                        __builtin_amdgcn_sched_barrier(0);
                        ++n;
                    }
                }
            }
        }
    };

    // ---- main loop ---------------------------------------------------------------------------------
    issue_copies(0);
#pragma unroll
    for (int i = 0; i < (BN == 256 ? 2 : 3); ++i) load_staged(st[i], min(i, steps1 - 1));
    if (nsteps > 1) issue_copies(1);
    // Pair table: a byte of codes (two adjacent k, low nibble first) selects the 8-byte entry
    // (c[lo], c[hi]) -- one LDS read dequantizes two weights.  The 256 entries are replicated 16 times,
    // entry b of replica q at b*128 + q*8, and lane l reads replica l & 15, so that lanes of one
    // 16-lane group never collide whatever their bytes are.
    {
        if (t < 16) reinterpret_cast<float*>(sT)[t] = d.cb.c[t];
        __syncthreads();
        const int b = t & 255;
        const float c_lo = reinterpret_cast<const float*>(sT)[b & 15], c_hi = reinterpret_cast<const float*>(sT)[b >> 4];
        __syncthreads();
        const float4 e = make_float4(c_lo, c_hi, c_lo, c_hi);
#pragma unroll
        for (int q = 0; q < 4; ++q) *reinterpret_cast<float4*>(sT + b * 128 + (t >> 8) * 64 + q * 16) = e;
        __syncthreads();
    }
    spread(st[0]);
#pragma unroll
    for (int u = 0; u < 4 * D; ++u) {
        lv[0][u & 3] = look_up(st[0], u);
        finish(st[0], u, lv[0], sW);
    }
    publish(Int<0>{});
    read_w(0, 0, wf[0]);
    read_x(0, 0, 0, xf[0]);
    if (steps1 > 1) {
#pragma unroll
        for (int u = 0; u < (BN == 256 ? 4 : 8); ++u) lv[u >> 2][u & 3] = look_up(st[1], u);
    }
    int s = 0;
    // (s is a multiple of the number of sets behind the first loop)
    if constexpr (BN == 128) {
        for (; s + 5 < steps1; s += 4) {
            step(Int<1>{}, Int<0>{}, s);
            step(Int<1>{}, Int<1>{}, s + 1);
            step(Int<1>{}, Int<2>{}, s + 2);
            step(Int<1>{}, Int<3>{}, s + 3);
        }
        for (; s < steps1; ++s) {
            step(Int<0>{}, Int<0>{}, s);
            st[1] = st[2]; st[2] = st[3];
        }
    } else {
        for (; s + 3 < steps1; s += 2) {
            step(Int<1>{}, Int<0>{}, s);
            step(Int<1>{}, Int<1>{}, s + 1);
        }
        for (; s < steps1; ++s) {
            step(Int<0>{}, Int<0>{}, s);
            st[1] = st[0];
        }
    }
    for (; s < nsteps; ++s) step(Int<2>{}, Int<0>{}, s);
    publish(Int<0>{});                                     // every wave is done reading the tiles

    // ---- epilogue ---------------------------------------------------------------------------------------
    // A lane holds features n..n+3 of one token per accumulator, i.e. 8 bytes of an output row.
    // The wave first lays its part out in LDS (the tiles are dead by now) as bf16 rows of
    // 128 bytes (pitch 144), then reads it back 16 bytes per lane so that every global store
    // instruction writes eight complete 128-byte row segments.
    {
        constexpr int kPitch = 144;
        const int el = lane_id(), er = el & 15, eg = el >> 4;
        unsigned char* eb = smem + wave * (16 * MB * kPitch);
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < MB; ++b) {
                uint2 o;
                o.x = pack_bf16(acc[a][b][0] * out_scale, acc[a][b][1] * out_scale);
                o.y = pack_bf16(acc[a][b][2] * out_scale, acc[a][b][3] * out_scale);
                *reinterpret_cast<uint2*>(eb + (b * 16 + er) * kPitch + (a * 16 + eg * 4) * 2) = o;
            }
        const int erow = el >> 3, echunk = el & 7;
        const int n = n0 + wn0 + echunk * 8;
#pragma unroll 8
        for (int i = 0; i < 2 * MB; ++i) {
            const int row = i * 8 + erow;
            const uint4 v = *reinterpret_cast<const uint4*>(eb + row * kPitch + echunk * 16);
            const int64_t m = m0 + wm0 + row;
            if (m < M && n < N) {
                typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
                const u32x4 vv = {v.x, v.y, v.z, v.w};
                __builtin_nontemporal_store(vv, reinterpret_cast<u32x4*>(C + m * ldc + n));
            }
        }
    }
}

template <int BN, bool BETA, int BR, bool TR>
int launch_cfg(const GemmDesc& d, hipStream_t st) {
    constexpr size_t smem = 2 * (kTileX + BN * 128) + kTableBytes;
    auto kern = k_qlinear<BN, BETA, BR, TR>;
    // set once per instantiation; the initialisation of a function-local static is thread safe
    static const bool attr_ok = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem) == hipSuccess;
    if (!attr_ok) return QBLORA_ERR_LAUNCH;
    int64_t tiles = ((d.M + BM - 1) / BM) * ((d.N + BN - 1) / BN);
    hipLaunchKernelGGL(kern, dim3((unsigned)tiles), dim3(kThreads), smem, st, d);
    return launch_status();
}

// Time of a launch in ns, by tile width: a k-step with every CU busy and with a few (a last round of workgroups, one per
// CU, lies in between: the clock holds up to about 3/4 of them).  256 x 128 tiles take 0.65 of the 256 x 256 tiles' time
// for half the work, so they pay where the wide ones leave more than a third of the CUs idle or start a round for a few
// tiles.  us on 256 x 256 / 256 x 128 tiles:
// 1024 x 4096 x 4096 105 / 71, 4096 x 4096 x 4096 124 / 141, 700 x 11008 x 4096 106 / 132, 512 x 11008 x 4096 105 / 69,
// 700 x 22016 x 8192 398 / 369, 2047 x 16384 x 8192 440 / 532, 4096 x 5120 x 13824 673 / 630.
struct Plan { bool wide; int64_t ns; };
Plan plan(int64_t M, int N, int64_t steps) {
    auto step_ns = [&](int bn, int64_t few, int64_t full) {
        const int64_t tiles = (M + BM - 1) / BM * ((N + bn - 1) / bn), last = tiles % 256;
        return tiles / 256 * full + (last ? few + (full - few) * last * last / 65536 : 0);
    };
    const int64_t wide = step_ns(256, 1490, 1840), narrow = step_ns(128, 950, 1080);
    return wide < narrow ? Plan{true, wide * steps} : Plan{false, narrow * steps};
}

template <bool BETA, int BR>
int launch_tile(const GemmDesc& d, hipStream_t st) {
    const bool wide = plan(d.M, d.N, 1).wide;
    if (d.qmode == 4) return wide ? launch_cfg<256, BETA, BR, true>(d, st) : launch_cfg<128, BETA, BR, true>(d, st);
    return wide ? launch_cfg<256, BETA, BR, false>(d, st) : launch_cfg<128, BETA, BR, false>(d, st);
}

}  // namespace

int64_t qlinear_ns(int64_t M, int N, int K) { return plan(M, N, K / kBK).ns; }

// The quantized GEMMs of the layer (qmode 1 and 4, bf16 output, no auxiliary outputs).
int launch_qlinear(const GemmDesc& d, hipStream_t st) {
    if (d.M <= 0 || d.N <= 0) return QBLORA_OK;
    if (d.out_f32 || d.C2 || d.C_lo) return QBLORA_ERR_UNSUPPORTED;
    if (d.qmode == 4 && (!d.scales || d.N != d.d_in || d.d_out % kBK != 0)) return QBLORA_ERR_UNSUPPORTED;
    if (d.block_rows == 8) {
        // 8 x 8 blocks ask for block parameters on a 16-byte boundary, here as everywhere; tile-ordered scales do not exist
        if (d.scales_tiled || !d.scales || d.d_out % 8 != 0 || (reinterpret_cast<uintptr_t>(d.scales) & 15) ||
            (reinterpret_cast<uintptr_t>(d.beta) & 15))
            return QBLORA_ERR_UNSUPPORTED;
        return d.beta ? launch_tile<true, 8>(d, st) : launch_tile<false, 8>(d, st);
    }
    if (d.qmode == 1 && !d.scales_tiled) return QBLORA_ERR_UNSUPPORTED;
    return d.beta ? launch_tile<true, 1>(d, st) : launch_tile<false, 1>(d, st);
}

}  // namespace qblora
