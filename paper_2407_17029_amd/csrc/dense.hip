// Contraction of the adapted layer on a weight that has been dequantized once (gfx950):
//
//   C[M,N] = X1[M,K1] * W1^T  +  X2[M,K2] * W2[N/div2, K2]^T          (bf16 operands, fp32 accumulation)
//
// W1 is the 16-bit compute weight of Eq. 1 in MFMA operand order (DequantDesc): the 16 bytes lane l
// of a wave needs for rows 16i .. 16i+15 and the 32-wide k slice j sit at ((i*(K1/32) + j)*64 + l)*16, so a piece
// of 1 KB is one copy instruction into LDS and one conflict-free ds_read_b128 out of it.  The second segment is
// the adapter's K-extension (forward: X2 = s*U, W2 = B^T with output row n using row n/lambda2; backward: X2 =
// dU/lambda1, W2 = A with row k/lambda1): its steps run through the same ring, W2's rows gathered by the copies.
//
// Bound: the matrix pipe.  Two kernels, by the size of the tile:
//
// k_dense, 256 x 256 tiles, for calls that fill rounds of the chip with them (1450 to 1510 TFLOP/s at 1.6-1.7 GHz, where the
// part is power-limited), sliced too, and for operands that outgrow the memory-side cache (dense_call_plan).  A workgroup is 8 wave64 as 2 (tokens) x 4 (features), two waves to a SIMD; a wave owns 128 tokens x
// 64 features.  The two waves of a SIMD belong to different halves of the workgroup (waves 0-3 and 4-7) that alternate
// strictly: while one half runs a compute phase (16 MFMAs, 16 cycles each) the other runs a memory phase (LDS fragment reads
// for its next compute phase, two copies into the ring, the waits), with a barrier between phases.  The second half passes one
// extra barrier at the start, so a compute phase always has a memory phase beside it: fragment reads, their latency and the
// refills hide under the other wave's MFMAs, and the copies leave evenly spread instead of in a burst behind a barrier.  The
// waits are exact counts: a part of a tile (16 KB, 2 copies a wave) is waited for at the end of the memory phase in front of
// the one that reads it, with 12 younger copies still in flight.  A region of the ring is refilled from the memory phase
// behind the one that read it: reads complete (lgkmcnt(0)) in front of the barrier that ends their phase, and the other half's
// same phase ends one barrier earlier than the refill starts.
//
// k_flow, smaller tiles.  Eight waves contract, four others, one to a SIMD, do nothing but copy: a copy
// instruction holds up the wave that issues it, and among the MFMAs that cost a quarter of the time.  The fragments of the next
// 64 or 32 wide step are read between the MFMAs of this one; one barrier a step says that the next stage is in and that the
// last one is free.  us in the phased form (which smaller tiles had too) / with the copies among the MFMAs / here: 1337 x 5120 x
// 5184 in 128 x 256 tiles 71 / 72 / 60, 1024 x 4096 x 4608 in 128 x 128 42.4 / 38.1 / 33.9 (without any copies: 28.6), 334 x 4224
// x 8064 64 / 52 / 45, 512 x 4096 x 11136 in four slices of 128 x 256 51 / 51 / 47.
//
// All copies are direct (global_load_lds, 16 bytes a lane) in assembly statements without register outputs, in program order.
// k is accumulated in ascending order by v_mfma_f32_16x16x32_bf16, as in the kernel that contracts from the codes
// (qlinear.hip), so all of them give the same bits where they are not sliced.
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace qblora {

namespace {

constexpr int kThreads = 512;
constexpr int kBK = 64;
constexpr int kPart = 16384;                      // bytes of a tile part: 128 token rows or 4 x 32 weight rows, 64 k

__device__ __align__(16) const uint32_t g_zero_chunk[4] = {0u, 0u, 0u, 0u};

__device__ __forceinline__ void copy16_to_lds(const void* src, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(lds_base), "v"(src) : "memory");
}
__device__ __forceinline__ void copy16_to_lds(const void* uniform_base, uint32_t lane_offset, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_base), "v"(lane_offset), "s"(uniform_base) : "memory");
}
__device__ __forceinline__ uint32_t lds_address(const void* p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

template <int N> using Int = std::integral_constant<int, N>;

// end of a memory phase: fragment reads done, at most N copies of this wave still in flight, then the barrier
template <int N>
__device__ __forceinline__ void end_memory(Int<N>) {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
    __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ void end_compute() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// 256 x 256 tiles
constexpr int MB = 4, NB = 2;                                               // a wave's 32-row blocks of tokens and features
struct Ring {
    static constexpr int kStages = 2;
    static constexpr int kX = MB * 8192, kW = NB * kPart, kStage = kX + kW;     // bytes
    static constexpr int kPitch = NB * 64 + 16;                                 // epilogue: output row of a wave in LDS
    static constexpr int kEpilogue = 8 * MB * 32 * kPitch;
    static constexpr int kLds = kStages * kStage > kEpilogue ? kStages * kStage : kEpilogue;
};

template <bool SLICED>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_dense(GemmDesc d) {
    using R = Ring;
    constexpr int BM = 64 * MB, BN = 128 * NB, S = R::kStages;
    extern __shared__ __align__(16) unsigned char smem[];

    const int64_t M = d.M;
    const int N = d.N, K2 = d.K2, div2 = d.div2;
    const int all_steps = d.K1 / kBK + (K2 + kBK - 1) / kBK;
    const int64_t ldx2 = d.ldx2, ldw2 = d.ldw2;
    const qblora_bf16* const X2 = d.X2;
    const qblora_bf16* const W2 = d.W2;

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const int r = lane & 15, g = lane >> 4;       // row of a 16-row operand block, group of 8 k

    // Tile assignment: workgroup ids go to the XCDs round-robin; each XCD gets a contiguous range of tiles, grouped
    // along tokens so that the tiles it runs at a time share token and weight panels in its L2.
    const int tiles_m = (int)((M + BM - 1) / BM), tiles_n = (N + BN - 1) / BN, ntiles = tiles_m * tiles_n;
    const int splits = SLICED ? d.splits : 1;
    int L;
    {
        const int units = ntiles * splits, xcd = blockIdx.x & 7, q = units >> 3, rem = units & 7;
        L = xcd * q + min(xcd, rem) + (blockIdx.x >> 3);
    }
    // slice z of the contraction (all tiles of a slice are neighbours): n steps from step0 on, at least one
    int z = 0, step0 = 0, n = all_steps;
    if constexpr (SLICED) {
        z = L / ntiles;
        step0 = all_steps * z / splits;
        n = all_steps * (z + 1) / splits - step0;
        L -= z * ntiles;
    }
    const int steps1 = d.K1 / kBK - step0;        // steps from here on that belong to the first segment (may be negative)
    constexpr int GM = 4;
    const int in_group = GM * tiles_n, first_m = (L / in_group) * GM, gsize = min(tiles_m - first_m, GM);
    const int64_t m0 = (int64_t)(first_m + (L % in_group) % gsize) * BM;
    const int n0 = (L % in_group) / gsize * BN;

    // ---- copies into the ring ---------------------------------------------------------------------------
    // Token part p: rows 64p .. 64p+63 of both wave rows' tokens; wave (wm, wn) copies 2 x 8 rows.  LDS rows are
    // 128 bytes with the 16-byte chunks XOR-swizzled by (row >> 1) & 7, applied by choosing which global chunk a
    // lane fetches.  (A ds_read_b128 is served 16 lanes at a time, lanes 0-3, 12-15 and 20-27 first: in the fragment
    // pattern those are 16 different rows, half of them with the neighbouring chunk, and this swizzle puts them in 16
    // different 16-byte bank groups.  With the (row ^ row >> 3) & 7 of the 32-row fragments of qlinear.hip they
    // collide in pairs: 19 % of the kernel's cycles.)
    uint32_t xoff[MB / 2][2];
    int xchunk[2];
    const qblora_bf16* const x_tile = d.X1 + m0 * d.ldx1 + (int64_t)step0 * kBK;
#pragma unroll
    for (int i = 0; i < 2; ++i) xchunk[i] = (lane & 7) ^ (4 * i + (lane >> 4));
    auto token_row = [&](int p, int i) __attribute__((always_inline)) {          // tile row, clamped to the last token
        const int row = wm * 32 * MB + p * 64 + 16 * wn + 8 * i + (lane >> 3);
        return m0 + row > M - 1 ? (int)(M - 1 - m0) : row;
    };
#pragma unroll
    for (int p = 0; p < MB / 2; ++p)
#pragma unroll
        for (int i = 0; i < 2; ++i) xoff[p][i] = (uint32_t)(token_row(p, i) * d.ldx1 * 2) + (uint32_t)(xchunk[i] << 4);
    // Weight part a: the a-th 32-row block of each wave column, 4 pieces of 1 KB each; wave w copies pieces 2w, 2w+1.
    const int blocks32 = (N + 31) / 32;
    const unsigned char* wbase[NB];
    int wblk[NB];
#pragma unroll
    for (int a = 0; a < NB; ++a) {
        wblk[a] = min(n0 / 32 + (wave >> 1) * NB + a, blocks32 - 1);    // rows past N: any block, results never stored
        wbase[a] = reinterpret_cast<const unsigned char*>(d.W1) + (int64_t)(2 * wblk[a] + (wave & 1)) * (d.K1 / 32) * 1024 + (int64_t)step0 * 2048;
    }
    const uint32_t lane16 = (uint32_t)lane * 16u;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem));
    const uint32_t lds_x = lds0 + (uint32_t)(wm * 32 * MB + 16 * wn) * 128u, lds_w = lds0 + R::kX + (uint32_t)wave * 2048u;

    auto issue_x = [&](int p, int step, uint32_t slot) __attribute__((always_inline)) {
        if (step < steps1) {
            const qblora_bf16* base = x_tile + step * kBK;
#pragma unroll
            for (int i = 0; i < 2; ++i) copy16_to_lds(base, xoff[p][i], lds_x + slot + p * 8192 + i * 1024);
        } else {
            const int k0 = (step - steps1) * kBK;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int k = k0 + xchunk[i] * 8;                       // chunks at or beyond K2 are zeros
                const qblora_bf16* src = X2 + (m0 + token_row(p, i)) * ldx2 + k;
                copy16_to_lds(k < K2 ? src : reinterpret_cast<const qblora_bf16*>(g_zero_chunk), lds_x + slot + p * 8192 + i * 1024);
            }
        }
    };
    auto issue_w = [&](int a, int step, uint32_t slot) __attribute__((always_inline)) {
        if (step < steps1) {
            const unsigned char* base = wbase[a] + (int64_t)step * 2048;
#pragma unroll
            for (int i = 0; i < 2; ++i) copy16_to_lds(base + i * 1024, lane16, lds_w + slot + a * kPart + i * 1024);
        } else {
            const int row = min(wblk[a] * 32 + 16 * (wave & 1) + r, N - 1);
            const qblora_bf16* src = W2 + (int64_t)((uint32_t)row / (uint32_t)div2) * ldw2;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int k = (step - steps1) * kBK + i * 32 + g * 8;
                copy16_to_lds(k < K2 ? src + k : reinterpret_cast<const qblora_bf16*>(g_zero_chunk),
                              lds_w + slot + a * kPart + i * 1024);
            }
        }
    };

    // ---- fragments and MFMAs ----------------------------------------------------------------------------
    f32x4 acc[2 * NB][2 * MB];                    // [16 features][16 tokens]
#pragma unroll
    for (int a = 0; a < 2 * NB; ++a)
#pragma unroll
        for (int b = 0; b < 2 * MB; ++b) acc[a][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    bf16x8 xf[4][2], wf[NB][2][2];
    // 16-token block b, slice ks of 32 k: row wm*32*MB + 16b + r, chunk 4ks + g, i.e. (xa ^ (ks << 6)) + 2048 b
    const uint32_t xa = (uint32_t)((wm * 32 * MB + r) * 128 + ((g ^ (r >> 1)) << 4));
    const uint32_t wa = (uint32_t)(R::kX + wn * 4096 + lane * 16);
    auto read_x = [&](int p, uint32_t slot) __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int b = 0; b < 4; ++b)
                xf[b][ks] = *reinterpret_cast<const bf16x8*>(smem + ((xa ^ (uint32_t)(ks << 6)) + slot) + (4 * p + b) * 2048);
    };
    auto read_w = [&](int a, uint32_t slot) __attribute__((always_inline)) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                wf[a][h][ks] = *reinterpret_cast<const bf16x8*>(smem + (wa + slot) + a * kPart + h * 2048 + ks * 1024);
    };
    // The barrier that ends a compute phase stands in front of its last MFMA: the other half's first MFMAs then
    // reach the pipe as it drains (interval 292 -> 283 cycles against 256 of MFMAs).  The raised priority makes the
    // last MFMA issue ahead of the other half's; without it this half's next memory phase starts late (the whole
    // kernel 20 % slower with the barrier two MFMAs early).
    auto compute = [&](int a, int p) __attribute__((always_inline)) {
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    if (ks == 1 && h == 1 && b == 3) {
                        __builtin_amdgcn_s_setprio(3);
                        end_compute();
                    }
                    acc[2 * a + h][4 * p + b] =
                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[a][h][ks], xf[b][ks], acc[2 * a + h][4 * p + b], 0, 0, 0);
                }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(0);
    };
    auto slot_of = [&](int step) __attribute__((always_inline)) { return (uint32_t)(step % S) * (uint32_t)R::kStage; };

    // Phases of step s (reads -> MFMAs; copies for step s+2 into the region read one phase earlier):
    //   0: X part 0 -> (W0, X0), W0(s+2);   1: W1 -> (W1, X0), X0(s+2);
    //   2: X part 1 -> (W0, X1), W1(s+2);   3: W0(s+1) -> (W1, X1), X1(s+2)
    issue_w(0, 0, 0); issue_x(0, 0, 0); issue_w(1, 0, 0); issue_x(1, 0, 0);
    if (n > 1) {
        issue_w(0, 1, R::kStage); issue_x(0, 1, R::kStage); issue_w(1, 1, R::kStage); issue_x(1, 1, R::kStage);
        end_memory(Int<12>{});
    } else {
        end_memory(Int<0>{});
    }
    read_w(0, 0);
    end_memory(Int<12>{});
    if (wm) end_compute();                                       // the second half runs one phase behind
    auto step = [&](int s, auto issue, auto last, auto w0, auto w1, auto w2, auto w3) __attribute__((always_inline)) {
        const uint32_t cur = slot_of(s), nxt = (uint32_t)R::kStage - cur;
        read_x(0, cur);
        if constexpr (issue.value) issue_w(0, s + 2, cur);
        end_memory(w0);
        compute(0, 0);
        read_w(1, cur);
        if constexpr (issue.value) issue_x(0, s + 2, cur);
        end_memory(w1);
        compute(1, 0);
        read_x(1, cur);
        if constexpr (issue.value) issue_w(1, s + 2, cur);
        end_memory(w2);
        compute(0, 1);
        if constexpr (!last.value) read_w(0, nxt);
        if constexpr (issue.value) issue_x(1, s + 2, cur);
        end_memory(w3);
        compute(1, 1);
    };
    int s = 0;
    for (; s + 2 < n; ++s) step(s, Int<1>{}, Int<0>{}, Int<12>{}, Int<12>{}, Int<12>{}, Int<12>{});
    if (s + 1 < n) {
        step(s, Int<0>{}, Int<0>{}, Int<10>{}, Int<8>{}, Int<6>{}, Int<4>{});
        ++s;
    }
    step(s, Int<0>{}, Int<1>{}, Int<2>{}, Int<0>{}, Int<0>{}, Int<0>{});
    if (!wm) end_compute();                                          // barriers even out
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");   // LDS is free: no copy under way, no wave reading

    // ---- epilogue -----------------------------------------------------------------------------------------
    if constexpr (SLICED) {                                          // partial sums: 4 features of one token per lane
        float* const part = d.part + (int64_t)z * M * N;
#pragma unroll
        for (int b = 0; b < 2 * MB; ++b) {
            const int64_t m = m0 + wm * 32 * MB + 16 * b + r;
#pragma unroll
            for (int a = 0; a < 2 * NB; ++a) {
                const int nn = n0 + wn * 32 * NB + 16 * a + 4 * g;
                if (m < M && nn < N) *reinterpret_cast<f32x4*>(part + m * N + nn) = acc[a][b];
            }
        }
        return;
    }
    // A lane holds features n..n+3 of one token per accumulator.  The wave lays its part out in LDS as bf16
    // rows and reads it back 16 bytes a lane, so that a store instruction writes whole row segments.
    {
        constexpr int kPitch = R::kPitch, kChunks = NB * 4, kRows = 64 / kChunks;
        qblora_bf16* const C = reinterpret_cast<qblora_bf16*>(d.C);
        const float out_scale = d.out_scale;
        unsigned char* eb = smem + wave * (MB * 32 * kPitch);
#pragma unroll
        for (int a = 0; a < 2 * NB; ++a)
#pragma unroll
            for (int b = 0; b < 2 * MB; ++b) {
                uint2 o;
                o.x = pack_bf16(acc[a][b][0] * out_scale, acc[a][b][1] * out_scale);
                o.y = pack_bf16(acc[a][b][2] * out_scale, acc[a][b][3] * out_scale);
                *reinterpret_cast<uint2*>(eb + (b * 16 + r) * kPitch + (a * 16 + g * 4) * 2) = o;
            }
        const int erow = lane / kChunks, echunk = lane % kChunks;
        const int nn = n0 + wn * 32 * NB + echunk * 8;
#pragma unroll 8
        for (int i = 0; i < MB * 32 / kRows; ++i) {
            const int row = i * kRows + erow;
            const int64_t m = m0 + wm * 32 * MB + row;
            typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
            const u32x4 v = *reinterpret_cast<const u32x4*>(eb + row * kPitch + echunk * 16);
            if (m < M && nn < N) __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(C + m * d.ldc + nn));
        }
    }
}

// Smaller tiles: BM tokens x BN features, WN of the eight contracting waves along the features.  A stage of the ring holds the
// token rows of a step, 128 bytes each, swizzled as above, and behind them the weight's pieces, 1 KB per 16 rows and 32-wide
// slice.  HALF: a fragment set is a 32-wide slice, and the barrier stands between a step's two; else a whole step (128 x 128
// tiles, whose eight MFMAs a slice would not cover the reads' latency: 34.8 -> 33.9 us).
template <int BM, int BN, int WN>
struct Flow {
    static constexpr int WM = 8 / WN, TB = BM / WM / 16, FB = BN / WN / 16;    // 16-row blocks of a wave
    static constexpr int kX = BM * 128, kStage = kX + BN * 128;                 // bytes
    static constexpr int kStages = 160 * 1024 / kStage;
    static constexpr int PX = BM / 32, PW = BN / 32, kOps = PX + PW;            // copies of a copying wave and step
    static constexpr int kPitch = FB * 32 + 16;
    static constexpr int kEpilogue = 8 * TB * 16 * kPitch;
    static constexpr int kLds = kStages * kStage > kEpilogue ? kStages * kStage : kEpilogue;
};

constexpr int kFlowThreads = 768;                                               // eight waves contract, four copy
template <int BM, int BN, int WN, bool HALF>
__global__ __launch_bounds__(kFlowThreads) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_flow(GemmDesc d) {
    using F = Flow<BM, BN, WN>;
    constexpr int TB = F::TB, FB = F::FB, S = F::kStages, PX = F::PX, PW = F::PW;
    extern __shared__ __align__(16) unsigned char smem[];
    const int64_t M = d.M;
    const int N = d.N, K2 = d.K2, div2 = d.div2;
    const int all_steps = d.K1 / kBK + (K2 + kBK - 1) / kBK;
    const int64_t ldx2 = d.ldx2, ldw2 = d.ldw2;
    const qblora_bf16* const X2 = d.X2;
    const qblora_bf16* const W2 = d.W2;
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int r = lane & 15, g = lane >> 4;

    const int tiles_m = (int)((M + BM - 1) / BM), tiles_n = (N + BN - 1) / BN, ntiles = tiles_m * tiles_n;
    const int splits = d.splits > 1 ? d.splits : 1;
    int L;
    {
        const int units = ntiles * splits, xcd = blockIdx.x & 7, q = units >> 3, rem = units & 7;
        L = xcd * q + min(xcd, rem) + (blockIdx.x >> 3);
    }
    int z = 0, step0 = 0, n = all_steps;
    if (splits > 1) {
        z = L / ntiles;
        step0 = all_steps * z / splits;
        n = all_steps * (z + 1) / splits - step0;
        L -= z * ntiles;
    }
    const int steps1 = d.K1 / kBK - step0;
    constexpr int GM = 4;
    const int in_group = GM * tiles_n, first_m = (L / in_group) * GM, gsize = min(tiles_m - first_m, GM);
    const int64_t m0 = (int64_t)(first_m + (L % in_group) % gsize) * BM;
    const int n0 = (L % in_group) / gsize * BN;

    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem));
    if (wave >= 8) {
        // copying wave c fills token rows 8*(PX*c + i) .. +7 and the weight pieces PW*c + i (16-row block p >> 1, 32-wide
        // slice p & 1)
        const int c = wave - 8;
        uint32_t xoff[PX];
        const qblora_bf16* const x_tile = d.X1 + m0 * d.ldx1 + (int64_t)step0 * kBK;
        auto token_row = [&](int i) __attribute__((always_inline)) {
            const int row = 8 * (PX * c + i) + (lane >> 3);
            return m0 + row > M - 1 ? (int)(M - 1 - m0) : row;
        };
        auto chunk_of = [&](int i) __attribute__((always_inline)) { return (lane & 7) ^ (4 * ((PX * c + i) & 1) + (lane >> 4)); };
#pragma unroll
        for (int i = 0; i < PX; ++i) xoff[i] = (uint32_t)(token_row(i) * d.ldx1 * 2) + (uint32_t)(chunk_of(i) << 4);
        int wblk[PW], wpiece[PW];                                       // 1 KB pieces from the weight's first: below 2^31
#pragma unroll
        for (int i = 0; i < PW; ++i) {
            const int p = PW * c + i;
            wblk[i] = min(n0 / 16 + (p >> 1), N / 16 - 1);              // rows past N: any block, results never stored
            wpiece[i] = __builtin_amdgcn_readfirstlane(wblk[i] * (d.K1 / 32) + step0 * 2 + (p & 1));
        }
        const unsigned char* const W1 = reinterpret_cast<const unsigned char*>(d.W1);
        const uint32_t lane16 = (uint32_t)lane * 16u;
        const uint32_t lds_x = lds0 + (uint32_t)c * (PX * 1024), lds_w = lds0 + F::kX + (uint32_t)c * (PW * 1024);
        auto issue = [&](int step, uint32_t slot) __attribute__((always_inline)) {
            if (step < steps1) {
#pragma unroll
                for (int i = 0; i < PX; ++i) copy16_to_lds(x_tile + step * kBK, xoff[i], lds_x + slot + i * 1024);
#pragma unroll
                for (int i = 0; i < PW; ++i) copy16_to_lds(W1 + (int64_t)(wpiece[i] + 2 * step) * 1024, lane16, lds_w + slot + i * 1024);
                return;
            }
            const int k0 = (step - steps1) * kBK;                       // chunks at or beyond K2 are zeros
#pragma unroll
            for (int i = 0; i < PX; ++i) {
                const int k = k0 + chunk_of(i) * 8;
                const qblora_bf16* src = X2 + (m0 + token_row(i)) * ldx2 + k;
                copy16_to_lds(k < K2 ? src : reinterpret_cast<const qblora_bf16*>(g_zero_chunk), lds_x + slot + i * 1024);
            }
#pragma unroll
            for (int i = 0; i < PW; ++i) {
                const qblora_bf16* src = W2 + (int64_t)((uint32_t)(wblk[i] * 16 + r) / (uint32_t)div2) * ldw2;
                const int k = k0 + ((PW * c + i) & 1) * 32 + g * 8;
                copy16_to_lds(k < K2 ? src + k : reinterpret_cast<const qblora_bf16*>(g_zero_chunk), lds_w + slot + i * 1024);
            }
        };
        // until at most `left` whole steps of this wave's copies are in flight
        auto landed = [&](int left) __attribute__((always_inline)) {
            if (left >= S - 2) asm volatile("s_waitcnt vmcnt(%0)" :: "n"((S - 2) * F::kOps) : "memory");
            else if (S > 3 && left == S - 3) asm volatile("s_waitcnt vmcnt(%0)" :: "n"((S > 3 ? S - 3 : 0) * F::kOps) : "memory");
            else if (S > 4 && left == S - 4) asm volatile("s_waitcnt vmcnt(%0)" :: "n"((S > 4 ? S - 4 : 0) * F::kOps) : "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        };
#pragma unroll 1
        for (int q = 0; q < S && q < n; ++q) issue(q, q * F::kStage);
        if (n >= S) asm volatile("s_waitcnt vmcnt(%0)" :: "n"((S - 1) * F::kOps) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        asm volatile("s_barrier" ::: "memory");                         // step 0 is in
        uint32_t slot = 0;
#pragma unroll 1
        for (int s = 0; s + 1 < n; ++s) {
            landed(n - 2 - s);
            asm volatile("s_barrier" ::: "memory");                     // step s + 1 is in, the stage of step s is free
            if (s + S < n) issue(s + S, slot);
            slot = slot + F::kStage == S * F::kStage ? 0u : slot + (uint32_t)F::kStage;
        }
        asm volatile("s_barrier" ::: "memory");
        return;
    }

    f32x4 acc[FB][TB];
#pragma unroll
    for (int a = 0; a < FB; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b) acc[a][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    constexpr int KS = HALF ? 1 : 2;                                 // 32-wide slices of a fragment set
    struct Frags { bf16x8 x[KS][TB], w[KS][FB]; };
    const uint32_t xa = (uint32_t)((wm * 16 * TB + r) * 128 + ((g ^ (r >> 1)) << 4));
    const uint32_t wa = (uint32_t)(F::kX + wn * FB * 2048 + lane * 16);
    constexpr int NR = KS * (TB + FB), NM = KS * TB * FB;
    auto read = [&](Frags& f, int i, int ks0, uint32_t slot) __attribute__((always_inline)) {        // fragment i of NR
        const int q = i / (TB + FB), ks = ks0 + q, j = i % (TB + FB);
        if (j < FB) f.w[q][j] = *reinterpret_cast<const bf16x8*>(smem + (wa + slot) + j * 2048 + ks * 1024);
        else f.x[q][j - FB] = *reinterpret_cast<const bf16x8*>(smem + ((xa ^ (uint32_t)(ks << 6)) + slot) + (j - FB) * 2048);
    };
    auto top = [&]() __attribute__((always_inline)) {                // this wave's reads are done; the next step is in
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    // the MFMAs of a set, and between them the reads of the next set
    auto contract = [&](const Frags& now, Frags& next, auto reads, int ks_next, uint32_t from) __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            const int q = m / (TB * FB), a = m / TB % FB, b = m % TB;
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(now.w[q][a], now.x[q][b], acc[a][b], 0, 0, 0);
            if constexpr (reads.value) {
#pragma unroll
                for (int i = m * NR / NM; i < (m + 1) * NR / NM; ++i) read(next, i, ks_next, from);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    uint32_t slot = 0;                                               // stage of the step in work
    auto next_slot = [&]() __attribute__((always_inline)) { return slot + F::kStage == S * F::kStage ? 0u : slot + (uint32_t)F::kStage; };
    asm volatile("s_barrier" ::: "memory");                          // step 0 is in
    Frags f0, f1;
#pragma unroll
    for (int i = 0; i < NR; ++i) read(f0, i, 0, 0);
    int s = 0;
    if constexpr (HALF) {
        // first slice: its MFMAs beside the reads of the second; the barrier; second slice beside the next step's first
        for (; s + 1 < n; ++s) {
            contract(f0, f1, Int<1>{}, 1, slot);
            top();
            contract(f1, f0, Int<1>{}, 0, next_slot());
            slot = next_slot();
        }
        contract(f0, f1, Int<1>{}, 1, slot);
        contract(f1, f0, Int<0>{}, 0, 0);
    } else {
        auto step = [&](const Frags& now, Frags& next) __attribute__((always_inline)) {
            top();
            contract(now, next, Int<1>{}, 0, next_slot());
            slot = next_slot();
        };
        for (; s + 2 < n; s += 2) { step(f0, f1); step(f1, f0); }
        if (s + 1 < n) { step(f0, f1); f0 = f1; }
        contract(f0, f1, Int<0>{}, 0, 0);
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");   // LDS is free: no copy under way, no wave reading

    if (splits > 1) {                                                // partial sums: 4 features of one token per lane
        float* const part = d.part + (int64_t)z * M * N;
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            const int64_t m = m0 + wm * 16 * TB + 16 * b + r;
#pragma unroll
            for (int a = 0; a < FB; ++a) {
                const int nn = n0 + wn * 16 * FB + 16 * a + 4 * g;
                if (m < M && nn < N) *reinterpret_cast<f32x4*>(part + m * N + nn) = acc[a][b];
            }
        }
        return;
    }
    {
        constexpr int kPitch = F::kPitch, kChunks = FB * 2, kTotal = TB * 16 * kChunks;
        qblora_bf16* const C = reinterpret_cast<qblora_bf16*>(d.C);
        const float out_scale = d.out_scale;
        unsigned char* eb = smem + wave * (TB * 16 * kPitch);
#pragma unroll
        for (int a = 0; a < FB; ++a)
#pragma unroll
            for (int b = 0; b < TB; ++b) {
                uint2 o;
                o.x = pack_bf16(acc[a][b][0] * out_scale, acc[a][b][1] * out_scale);
                o.y = pack_bf16(acc[a][b][2] * out_scale, acc[a][b][3] * out_scale);
                *reinterpret_cast<uint2*>(eb + (b * 16 + r) * kPitch + (a * 16 + g * 4) * 2) = o;
            }
#pragma unroll 8
        for (int i = lane; i < kTotal; i += 64) {
            const int row = i / kChunks, echunk = i % kChunks;
            const int nn = n0 + wn * 16 * FB + echunk * 8;
            const int64_t m = m0 + wm * 16 * TB + row;
            typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
            const u32x4 v = *reinterpret_cast<const u32x4*>(eb + row * kPitch + echunk * 16);
            if (m < M && nn < N) __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(C + m * d.ldc + nn));
        }
    }
}

// The slices' partial sums added in slice order, eight features of one token per thread.
__global__ __launch_bounds__(256) void k_dense_reduce(GemmDesc d) {
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8, plane = d.M * d.N;
    if (i >= plane) return;
    f32x4 lo = {0.0f, 0.0f, 0.0f, 0.0f}, hi = lo;
    for (int z0 = 0; z0 < d.splits; z0 += 4) {
        f32x4 v[4][2];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const f32x4* src = reinterpret_cast<const f32x4*>(d.part + min(z0 + u, d.splits - 1) * plane + i);
            v[u][0] = src[0]; v[u][1] = src[1];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (z0 + u < d.splits) { lo += v[u][0]; hi += v[u][1]; }
    }
    const int64_t m = i / d.N;
    const float s = d.out_scale;
    *reinterpret_cast<uint4*>(reinterpret_cast<qblora_bf16*>(d.C) + m * d.ldc + (i - m * d.N)) =
        make_uint4(pack_bf16(lo[0] * s, lo[1] * s), pack_bf16(lo[2] * s, lo[3] * s),
                   pack_bf16(hi[0] * s, hi[1] * s), pack_bf16(hi[2] * s, hi[3] * s));
}

template <typename K>
int launch_tiles(K kern, bool lds_ok, int smem, int threads, int bm, int bn, const GemmDesc& d, hipStream_t st) {
    if (!lds_ok) return QBLORA_ERR_LAUNCH;
    const int64_t tiles = ((d.M + bm - 1) / bm) * ((d.N + bn - 1) / bn);
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles * (d.splits > 1 ? d.splits : 1))), dim3(threads), smem, st, d);
    if (d.splits > 1)
        hipLaunchKernelGGL(k_dense_reduce, dim3((unsigned)((d.M * d.N / 8 + 255) / 256)), dim3(256), 0, st, d);
    return launch_status();
}

// set once per kernel; callers keep the result in a function-local static, whose initialisation is thread safe
template <typename K>
bool set_lds(K kern, int smem) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, smem) == hipSuccess;
}

template <bool SLICED>
int launch_large(const GemmDesc& d, hipStream_t st) {
    static const bool ok = set_lds(k_dense<SLICED>, Ring::kLds);
    return launch_tiles(k_dense<SLICED>, ok, Ring::kLds, kThreads, 64 * MB, 128 * NB, d, st);
}

template <int BM, int BN, int WN, bool HALF>
int launch_flow(const GemmDesc& d, hipStream_t st) {
    constexpr int smem = Flow<BM, BN, WN>::kLds;
    static const bool ok = set_lds(k_flow<BM, BN, WN, HALF>, smem);
    return launch_tiles(k_flow<BM, BN, WN, HALF>, ok, smem, kFlowThreads, BM, BN, d, st);
}

}  // namespace

// The most slices of a call, which workspaces count on, and the line between this form and the one from the codes on large
// weights: estimates by the times of the kernels that these were measured with, 256 x 256, 128 x 256, 256 x 128 and 128 x 128
// tiles.  `full` is the time of a k-step with every CU busy, `few` with a few, both in ns; a last round of workgroups (256, one
// per CU) that is not full lies in between.  A slice adds its fp32 partial tile, written and read once, and all of them the
// second launch.  What a call takes: dense_call_plan.
DensePlan dense_plan(int64_t M, int N, int k1, int k2, int max_splits) {
    struct Shape { int bm, bn; int64_t few, full; };
    static constexpr Shape shapes[4] = {{256, 256, 940, 1460}, {128, 256, 800, 920}, {256, 128, 800, 930}, {128, 128, 490, 570}};
    const int64_t steps = k1 / kBK + (k2 + kBK - 1) / kBK;
    DensePlan best{0, 1, INT64_MAX};
    for (int i = 0; i < 4; ++i) {
        const int64_t tiles = ((M + shapes[i].bm - 1) / shapes[i].bm) * ((N + shapes[i].bn - 1) / shapes[i].bn);
        for (int s = 1; s <= max_splits && (s == 1 || (tiles * s <= 256 && steps >= 4 * s)); ++s) {
            const int64_t units = tiles * s, last = units % 256;
            const int64_t step_ns = units / 256 * shapes[i].full +
                                    (last ? shapes[i].few + (shapes[i].full - shapes[i].few) * last / 256 : 0);
            int64_t t = step_ns * ((steps + s - 1) / s) * 4000;  // in ns / 4000: exactly linear in M while the tiles stay
            if (s > 1) t += 5000 * 4000 + M * N * 8 * s;         // bytes at 4 TB/s
            if (t < best.ns) best = DensePlan{i, s, t};
        }
    }
    best.ns /= 4000;
    return best;
}

// The tile and the slices of a call, by the present kernels' times: as above, but a last round of f of the 256 workgroups lies
// f^3 of the way from few to full (the clock holds to about half of them), and a round starts and ends in 1.6 us and what its
// output tiles take.  Larger tiles move fewer bytes per MFMA, which counts above all where the operands outgrow the memory-side
// cache (256 MB): the second pair of times, reached in steps between 180 and 285 MB.  Fitted to 1333 shapes of 16 to 9000 tokens, each
// timed in every tile and number of slices: a call on 257 tokens or more takes 0.9 % longer than in its best form on average, 4 % of
// them more than 6 %; fewer tokens 4 % on average.  With one pair of times, from weights of 9 to 47 million alone, 2921 x 12416 x 13120
// took 128 x 192 tiles, 1013 us with the pass over the weight, now 878; 698 x 4160 x 22720 unsliced 128 x 128 ones, 244, now five
// slices of 256 x 256, 179.  us for 256 x 256 / 128 x 256 / 128 x 192 / 192 x 192 / 128 x 128 tiles: 1337 x 5120 x 5184 99 / 60 / 86 /
// 59 / 71; 512 x 11008 x 4224 71 / 42 / 39 / 46 / 54; 1024 x 4096 x 4608 79 / 43 / 38 / 48 / 34; 334 x 4224 x 8064 128 / 67 / 53 / 75 /
// 45; 2048 x 4096 x 4224 81 / 53 / 71 / 58 / 61; 8192 x 5120 x 5184 315 / 313 / 346 / 330 / -; 8192 x 22016 x 8448 2032 / 2380 / 2592 /
// 2341 / -.
DensePlan dense_call_plan(int64_t M, int N, int k1, int k2, int max_splits) {
    struct Shape { int bm, bn; int64_t few, full, few_far, full_far; };
    static constexpr Shape shapes[7] = {{256, 256, 940, 1310, 1070, 1440}, {128, 256, 490, 730, 985, 825}, {256, 128, 495, 735, 860, 850},
                                        {128, 128, 293, 421, 628, 554}, {128, 192, 386, 587, 814, 682}, {192, 128, 383, 574, 653, 685},
                                        {192, 192, 545, 824, 815, 843}};
    const int64_t steps = k1 / kBK + (k2 + kBK - 1) / kBK, far = std::min<int64_t>(std::max<int64_t>(((M + N) * k1 >> 19) - 180, 0), 105);
    const int most = max_splits > 1 ? dense_plan(M, N, k1, k2, max_splits).splits : 1;
    DensePlan best{0, 1, INT64_MAX};
    for (int i = 0; i < 7; ++i) {
        const Shape& c = shapes[i];
        const int64_t tiles = ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
        const int64_t few = c.few + (c.few_far - c.few) * far / 105, full = c.full + (c.full_far - c.full) * far / 105;
        for (int s = 1; s <= most && (s == 1 || (tiles * s <= 256 && steps >= 4 * s)); ++s) {
            const int64_t units = tiles * s, last = units % 256;
            const int64_t step_ns = units / 256 * full + (last ? few + (full - few) * (last * last * last) / (256 * 256 * 256) : 0);
            int64_t t = step_ns * ((steps + s - 1) / s) + (1600 + 75 * c.bm * c.bn / 1024) * ((units + 255) / 256);
            // (slices start far apart in both operands; their partial tiles stay in the caches: 10 TB/s)
            if (s > 1) t += t / 20 + 3500 + M * N * 8 * s / 10000;
            if (t < best.ns) best = DensePlan{i, s, t};
        }
    }
    return best;
}

// Tiles are counted in 128 or 256 tokens, so between two multiples of 128 every form's time is linear in M, with a slope
// that grows with its slices: the cheapest form's slices do not increase with M there, and each run of the same number
// has its most rows at its end.
int64_t dense_part_rows(int64_t M, int N, int k1, int k2) {
    if (M <= 0 || N <= 0) return 0;
    auto splits = [&](int64_t m) { return N % 8 != 0 ? 1 : (int64_t)dense_plan(m, N, k1, k2, 8).splits; };
    int64_t top = 0;                                             // the largest M whose tiles leave room for two slices
    for (const int bm : {128, 256})
        for (const int bn : {128, 256}) top = std::max<int64_t>(top, (int64_t)bm * (128 / ((N + bn - 1) / bn)));
    int64_t rows = 0;
    for (int64_t hi = std::min(M, top); hi > 0 && 8 * hi > rows; hi = (hi - 1) / 128 * 128) {
        const int64_t lo = (hi - 1) / 128 * 128 + 1, most = splits(lo);
        for (int64_t b = hi, s = splits(b); ; ) {
            if (s > 1) rows = std::max(rows, s * b);
            if (most <= s || most * b <= rows) break;
            int64_t more = lo, same = b;                         // the last M with more slices
            while (same - more > 1) {
                const int64_t mid = (more + same) / 2;
                if (splits(mid) > s) more = mid; else same = mid;
            }
            b = more;
            s = splits(b);
        }
    }
    return rows;
}

namespace {

// The 16-bit weight stays in the 256 MB memory-side cache between the pass and the contraction
bool weight_stays(int64_t N, int k1) { return N * k1 * 2 < (int64_t)256 << 20; }

}  // namespace

// The one-off pass takes 0.46 to 0.5 us per million weights, in a launch that both forms have (the re-layouts' or the narrow
// GEMM's sums'); the kernel from the codes wins on wide layers with few tokens.  us from the codes / dequantized first, without
// adapter: 512 x 22016 x 8192 223 / 264, 512 x 16384 x 8192 150 / 201, 1024 x 16384 x 8192 249 / 251, 650 x 8192 x 22016 363 / 361, 512 x
// 4096 x 4096 72 / 37, 512 x 11008 x 4096 77 / 64, 2048 x 22016 x 8192 680 / 616.  On weights whose 16-bit form outgrows the memory-side
// cache the first line stands alone, with the figures of dense_plan: those of dense_call_plan would send 560 to 740 x 8192 x 22016
// the other way (337 to 363 / 361 to 370), though 560 x 28672 x 8192 rightly (415 / 365).  Over 314 shapes near the line a call takes
// 0.8 % longer than the faster way on average, 1.0 % on those weights.
bool dense_pays(int64_t M, int N, int k1, int k2) {
    const int64_t codes = qlinear_ns(M, N, k1 + (k2 + kBK - 1) / kBK * kBK), weights = (int64_t)N * k1;
    const int64_t first = dense_plan(M, N, k1, k2, 1).ns + weights * 46 / 100000 + 2000;
    if (codes + 2000 >= first - first * 5 / 100) return true;
    return weight_stays(N, k1) && codes >= dense_call_plan(M, N, k1, k2, 1).ns + weights * 50 / 100000;
}

// The transposed weight's pass takes 0.62 us per million weights with the gradients' sums, and its contraction may be sliced,
// which the one from the codes is not.  us from the codes / dequantized first, M x N x K, without adapter: 64 x 22016 x 8192 127 / 176,
// 256 123 / 209, 512 198 / 268, 700 406 / 317; 700 x 8192 x 8192 142 / 108; 512 x 4096 x 11008 169 / 73; 512 x 11008 x 4096 72 / 61.  On
// large weights a margin of 10 %: with the slices' times of dense_plan, 5 % lost 6 and 10 % on two of 480 measured calls, 10 % on
// none.  Over 86 shapes near the line a call takes 2.1 % longer than the faster way on average, mostly for few tokens of wide
// layers (126 x 17280 x 9664 151 / 181, and dequantized first).
bool dense_pays_t(int64_t M, int N, int k1, int k2) {
    const int64_t codes = qlinear_ns(M, N, k1 + (k2 + kBK - 1) / kBK * kBK), weights = (int64_t)N * k1;
    const int64_t first = dense_plan(M, N, k1, k2, 8).ns + weights * 46 / 100000 + 2000;
    if (codes + 2000 >= first - first * 10 / 100) return true;
    return weight_stays(N, k1) && codes >= dense_call_plan(M, N, k1, k2, 8).ns + weights * 62 / 100000;
}

int dense_splits(int64_t M, int N, int k1, int k2) {
    if (M <= 0 || N <= 0 || N % 8 != 0) return 1;
    return dense_call_plan(M, N, k1, k2, 8).splits;
}

int launch_dense(const GemmDesc& d, hipStream_t st) {
    if (d.M <= 0 || d.N <= 0) return QBLORA_OK;
    // whole 64-wide steps of 16-byte chunks, whole 32-row blocks
    if (d.out_f32 || d.C2 || d.C_lo || !d.W1 || d.K1 <= 0 || d.K1 % kBK != 0 || d.N % 32 != 0 ||
        (reinterpret_cast<uintptr_t>(d.W1) & 15))
        return QBLORA_ERR_UNSUPPORTED;
    const DensePlan p = dense_call_plan(d.M, d.N, d.K1, d.K2, d.splits > 1 ? 8 : 1);
    if (d.splits > 1 && p.splits != d.splits) return QBLORA_ERR_UNSUPPORTED;       // not what dense_splits said
    switch (p.shape) {
        case 0: return d.splits > 1 ? launch_large<true>(d, st) : launch_large<false>(d, st);
        case 1: return launch_flow<128, 256, 4, true>(d, st);
        case 2: return launch_flow<256, 128, 2, true>(d, st);
        case 3: return launch_flow<128, 128, 4, false>(d, st);
        case 4: return launch_flow<128, 192, 4, true>(d, st);
        case 5: return launch_flow<192, 128, 2, true>(d, st);
        default: return launch_flow<192, 192, 4, true>(d, st);
    }
}

}  // namespace qblora
