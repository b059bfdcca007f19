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
// Bound: the matrix pipe.  A workgroup is 8 wave64 as 2 (tokens) x 4 (features), two waves to a SIMD; a wave owns
// 32*MB tokens x 32*NB features.  The two waves of a SIMD belong to different halves of the workgroup (waves 0-3
// and 4-7) that alternate strictly: while one half runs a compute phase (16 or 32 MFMAs, 16 cycles each) the other runs a
// memory phase (LDS fragment reads for its next compute phase, two to six copies into the ring, the waits), with
// a barrier between phases.  The second half passes one extra barrier at the start, so a compute phase always has
// a memory phase beside it: fragment reads, their latency and the refills hide under the other wave's MFMAs, and
// the copies leave evenly spread instead of in a burst behind a barrier.
//
// All copies are direct (global_load_lds, 16 bytes a lane) in assembly statements without register outputs, in
// program order, so the waits are exact counts: a part of a tile (16 KB, 2 copies a wave) is waited for at the end
// of the memory phase in front of the one that reads it, with 12 younger copies (8 in the smallest tile, 6 in the 128 x 256 one's long phases) still
// in flight.  A region of the ring is refilled from the memory phase behind the one that read it: reads complete
// (lgkmcnt(0)) in front of the barrier that ends their phase, and the other half's same phase ends one barrier
// earlier than the refill starts.
//
// k is accumulated in ascending order by v_mfma_f32_16x16x32_bf16, as in the kernel that contracts from the codes
// (qlinear.hip), so both give the same bits where this one is not sliced.
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

template <int MB, int NB>
struct Ring {
    static constexpr int kStages = MB == 4 && NB == 2 ? 2 : MB == 2 && NB == 1 ? 4 : 3;
    static constexpr int kX = MB * 8192, kW = NB * kPart, kStage = kX + kW;     // bytes
    static constexpr int kPitch = NB * 64 + 16;                                 // epilogue: output row of a wave in LDS
    static constexpr int kEpilogue = 8 * MB * 32 * kPitch;
    static constexpr int kLds = kStages * kStage > kEpilogue ? kStages * kStage : kEpilogue;
};

// WHOLE: a phase works on a whole step (128 x 256 tiles only)
template <int MB, int NB, bool WHOLE>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_dense(GemmDesc d) {
    using R = Ring<MB, NB>;
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
    const int splits = d.splits > 1 ? d.splits : 1;
    int L;
    {
        const int units = ntiles * splits, xcd = blockIdx.x & 7, q = units >> 3, rem = units & 7;
        L = xcd * q + min(xcd, rem) + (blockIdx.x >> 3);
    }
    // slice z of the contraction (all tiles of a slice are neighbours): n steps from step0 on, at least one
    int z = 0, step0 = 0, n = all_steps;
    if (splits > 1) {
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
    auto compute = [&](int a, int p, auto ends_phase) __attribute__((always_inline)) {
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    if (ends_phase.value && ks == 1 && h == 1 && b == 3) {
                        __builtin_amdgcn_s_setprio(3);
                        end_compute();
                    }
                    acc[2 * a + h][4 * p + b] =
                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[a][h][ks], xf[b][ks], acc[2 * a + h][4 * p + b], 0, 0, 0);
                }
        __builtin_amdgcn_sched_barrier(0);
        if (ends_phase.value) __builtin_amdgcn_s_setprio(0);
    };
    auto slot_of = [&](int step) __attribute__((always_inline)) { return (uint32_t)(step % S) * (uint32_t)R::kStage; };

    if constexpr (MB == 4 && NB == 2) {
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
            compute(0, 0, Int<1>{});
            read_w(1, cur);
            if constexpr (issue.value) issue_x(0, s + 2, cur);
            end_memory(w1);
            compute(1, 0, Int<1>{});
            read_x(1, cur);
            if constexpr (issue.value) issue_w(1, s + 2, cur);
            end_memory(w2);
            compute(0, 1, Int<1>{});
            if constexpr (!last.value) read_w(0, nxt);
            if constexpr (issue.value) issue_x(1, s + 2, cur);
            end_memory(w3);
            compute(1, 1, Int<1>{});
        };
        int s = 0;
        for (; s + 2 < n; ++s) step(s, Int<1>{}, Int<0>{}, Int<12>{}, Int<12>{}, Int<12>{}, Int<12>{});
        if (s + 1 < n) {
            step(s, Int<0>{}, Int<0>{}, Int<10>{}, Int<8>{}, Int<6>{}, Int<4>{});
            ++s;
        }
        step(s, Int<0>{}, Int<1>{}, Int<2>{}, Int<0>{}, Int<0>{}, Int<0>{});
    } else if constexpr (MB == 2 && NB == 2 && !WHOLE) {
        // 0: X -> (W0, X), W0(s+S) and W1(s+S-1);   1: W1, W0(s+1) -> (W1, X), X(s+S)
#pragma unroll
        for (int q = 0; q < S; ++q)
            if (q < n) {
                issue_w(0, q, q * R::kStage);
                if (q > 0) issue_w(1, q - 1, (q - 1) * R::kStage);
                issue_x(0, q, q * R::kStage);
            }
        if (n >= S) end_memory(Int<12>{});
        else { issue_w(1, n - 1, (n - 1) * R::kStage); end_memory(Int<0>{}); }
        read_w(0, 0);
        end_memory(Int<12>{});
        if (wm) end_compute();
        auto step = [&](int s, auto issue, auto wait) __attribute__((always_inline)) {
            const uint32_t cur = slot_of(s);
            read_x(0, cur);
            if constexpr (issue.value == 2) issue_w(0, s + S, cur);
            if constexpr (issue.value >= 1) issue_w(1, s + S - 1, slot_of(s + S - 1));
            end_memory(wait);
            compute(0, 0, Int<1>{});
            read_w(1, cur);
            if (issue.value == 2 || s + 1 < n) read_w(0, slot_of(s + 1));
            if constexpr (issue.value == 2) issue_x(0, s + S, cur);
            end_memory(wait);
            compute(1, 0, Int<1>{});
        };
        int s = 0;
        for (; s + S < n; ++s) step(s, Int<2>{}, Int<12>{});
        if (n >= S) step(s++, Int<1>{}, Int<0>{});
        for (; s < n; ++s) step(s, Int<0>{}, Int<0>{});
    } else if constexpr (MB == 2 && NB == 2) {
        // One phase of 32 MFMAs a step: X, W0, W1 -> all four, copies of step s+2 into the stage read a step earlier (the
        // other half's read of it ended one barrier ago).  Half as many barriers and waits for fragments as with a phase
        // for each of W0 and W1: 80 tiles of 5120 inputs 65 -> 56 us, 220 tiles 79 -> 74.  (256 x 128 tiles read 20
        // fragments for a step, and there the long phase is the slower one: 75.3 -> 77.9 us a call.)  Six copies instead
        // of twelve are in flight, though, which costs 1 to 2 us where slices fill the chip (see launch_dense).
        constexpr int kOps = 6;                                      // copies of a wave and step
#pragma unroll
        for (int q = 0; q < S - 1; ++q)
            if (q < n) { issue_x(0, q, q * R::kStage); issue_w(0, q, q * R::kStage); issue_w(1, q, q * R::kStage); }
        if (n >= S - 1) end_memory(Int<kOps * (S - 2)>{}); else end_memory(Int<0>{});
        if (wm) end_compute();
        auto step = [&](int s, auto issue, auto wait) __attribute__((always_inline)) {
            const uint32_t cur = slot_of(s);
            read_w(0, cur);
            read_w(1, cur);
            read_x(0, cur);
            if constexpr (issue.value) {
                const uint32_t to = slot_of(s + S - 1);
                issue_x(0, s + S - 1, to); issue_w(0, s + S - 1, to); issue_w(1, s + S - 1, to);
            }
            end_memory(wait);
            compute(0, 0, Int<0>{});
            compute(1, 0, Int<1>{});
        };
        int s = 0;
        for (; s + S - 1 < n; ++s) step(s, Int<1>{}, Int<kOps * (S - 2)>{});
        for (; s < n; ++s) step(s, Int<0>{}, Int<0>{});
    } else if constexpr (MB == 4 && NB == 1) {
        // 0: X part 0, W -> (W, X0), X1(s+S-1);   1: X part 1 -> (W, X1), X0(s+S) and W(s+S)
#pragma unroll
        for (int q = 0; q < S; ++q)
            if (q < n) {
                if (q > 0) issue_x(1, q - 1, (q - 1) * R::kStage);
                issue_x(0, q, q * R::kStage);
                issue_w(0, q, q * R::kStage);
            }
        if (n >= S) end_memory(Int<12>{});
        else { issue_x(1, n - 1, (n - 1) * R::kStage); end_memory(Int<0>{}); }
        if (wm) end_compute();
        auto step = [&](int s, auto issue, auto wait) __attribute__((always_inline)) {
            const uint32_t cur = slot_of(s);
            read_w(0, cur);
            read_x(0, cur);
            if constexpr (issue.value >= 1) issue_x(1, s + S - 1, slot_of(s + S - 1));
            end_memory(wait);
            compute(0, 0, Int<1>{});
            read_x(1, cur);
            if constexpr (issue.value == 2) { issue_x(0, s + S, cur); issue_w(0, s + S, cur); }
            end_memory(wait);
            compute(0, 1, Int<1>{});
        };
        int s = 0;
        for (; s + S < n; ++s) step(s, Int<2>{}, Int<12>{});
        if (n >= S) step(s++, Int<1>{}, Int<0>{});
        for (; s < n; ++s) step(s, Int<0>{}, Int<0>{});
    } else {
        // one phase a step: X, W -> MFMAs, copies of step s+S-1
#pragma unroll
        for (int q = 0; q < S - 1; ++q)
            if (q < n) { issue_x(0, q, q * R::kStage); issue_w(0, q, q * R::kStage); }
        if (n >= S - 1) end_memory(Int<4 * (S - 2)>{}); else end_memory(Int<0>{});
        if (wm) end_compute();
        auto step = [&](int s, auto issue, auto wait) __attribute__((always_inline)) {
            const uint32_t cur = slot_of(s);
            read_w(0, cur);
            read_x(0, cur);
            if constexpr (issue.value) {
                const uint32_t to = slot_of(s + S - 1);
                issue_x(0, s + S - 1, to); issue_w(0, s + S - 1, to);
            }
            end_memory(wait);
            compute(0, 0, Int<1>{});
        };
        int s = 0;
        for (; s + S - 1 < n; ++s) step(s, Int<1>{}, Int<4 * (S - 2)>{});
        for (; s < n; ++s) step(s, Int<0>{}, Int<0>{});
    }
    if (!wm) end_compute();                                          // barriers even out
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");   // LDS is free: no copy under way, no wave reading

    // ---- epilogue -----------------------------------------------------------------------------------------
    if (splits > 1) {                                                // partial sums: 4 features of one token per lane
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

template <int MB, int NB, bool WHOLE = false>
int launch_cfg(const GemmDesc& d, hipStream_t st) {
    auto kern = k_dense<MB, NB, WHOLE>;
    constexpr int smem = Ring<MB, NB>::kLds;
    // set once per instantiation; the initialisation of a function-local static is thread safe
    static const bool attr_ok = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                    hipFuncAttributeMaxDynamicSharedMemorySize, smem) == hipSuccess;
    if (!attr_ok) return QBLORA_ERR_LAUNCH;
    const int64_t tiles = ((d.M + 64 * MB - 1) / (64 * MB)) * ((d.N + 128 * NB - 1) / (128 * NB));
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles * (d.splits > 1 ? d.splits : 1))), dim3(kThreads), smem, st, d);
    if (d.splits > 1)
        hipLaunchKernelGGL(k_dense_reduce, dim3((unsigned)((d.M * d.N / 8 + 255) / 256)), dim3(256), 0, st, d);
    return launch_status();
}

}  // namespace

// Tile shape (and slices) by the estimated time.  `full` is the measured time of a k-step with every CU busy, `few`
// with a few (the clock is power-limited: 1.5-1.7 GHz with all matrix pipes busy, 2.4 with few), both in ns; a last
// round of workgroups (256, one per CU) that is not full lies in between.  (128 x 256 takes 690 and 870 since its phases
// hold a whole step; the choices below were measured with the older figures, which stay.)  Larger tiles move fewer bytes per MFMA
// (256 x 256 runs at 0.82-0.89 of the matrix pipe, 128 x 256 at 0.61, 128 x 128 at 0.40, where waves wait 0.42 of the time, LDS
// reads take 0.31 and copies 25 bytes a cycle) and need more tiles to fill the chip.  T x N x K, us for 256x256 / 128x256 / 256x128 / 128x128: 512 x 4096 x 11008 179 / 130 /
// 131 / 87; 512 x 11008 x 4096 77 / 61 / 60 / 76; 1337 x 5120 x 5120 94 / 71 / 74 / 90; 2500 x 5120 x 13824 263 / 350 /
// 358 / 439; 8192 x 4096 x 4096 192 / 233 / 238 / 285.  A slice adds its fp32 partial tile, written and read once, and
// all of them the second launch: 512 x 4096 x 11008 91 -> 54 + 7 us (128 x 256, four slices), 300 x 2048 x 6144 51 ->
// 19 + 4 (five), 128 x 4096 x 4096 35 -> 14 + 5 (five).
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

// Tiles are counted in 128 or 256 tokens, so between two multiples of 128 every form's time is linear in M, with a slope
// that grows with its slices: the cheapest form's slices do not increase with M there, and each run of the same number
// has its most rows at its end.
int64_t dense_part_rows(int64_t M, int N, int k1, int k2) {
    if (M <= 0 || N <= 0) return 0;
    auto splits = [&](int64_t m) { return (int64_t)dense_splits(m, N, k1, k2); };
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

// The one-off pass takes 0.46 us per million weights and a launch, which the forward's kernel from the codes does not
// spend (the launch is the re-layouts' by now, which both have; the line was measured with one of its own); that one wins on
// wide layers with few tokens.  us from the codes / dequantized first: 512 x 22016 x 8192 190 / 265,
// 512 x 16384 x 8192 138 / 194, 512 x 11008 x 4096 72 / 77, 1024 x 16384 x 8192 233 / 257, 512 x 4096 x 4096 70 / 46,
// 2048 x 22016 x 8192 632 / 610.  The margin of 5 % is for the estimates' errors: without it 72 of 1134 measured calls
// lose up to 9 % of their time, with it three lose 3 % (and 207 gain 17 % on average).
bool dense_pays(int64_t M, int N, int k1, int k2) {
    const int64_t first = dense_plan(M, N, k1, k2, 1).ns + (int64_t)N * k1 * 46 / 100000 + 2000;
    return qlinear_ns(M, N, k1 + (k2 + kBK - 1) / kBK * kBK) + 2000 >= first - first * 5 / 100;
}

// The transposed weight's pass is the same; its contraction may be sliced, which the one from the codes is not.  us from
// the codes / dequantized first, 8192 x 22016: 64 tokens 122 / 185, 256 122 / 223, 512 195 / 275, 700 376 / 401; 4096 x 11008
// at 512 67 / 76; 8192 x 8192 at 700 131 / 124.  A margin of 10 %: the slices' time is the less certain (with 5 % two of
// 480 measured calls lose 6 and 10 %, with 10 % none).
bool dense_pays_t(int64_t M, int N, int k1, int k2) {
    const int64_t first = dense_plan(M, N, k1, k2, 8).ns + (int64_t)N * k1 * 46 / 100000 + 2000;
    return qlinear_ns(M, N, k1 + (k2 + kBK - 1) / kBK * kBK) + 2000 >= first - first * 10 / 100;
}

int dense_splits(int64_t M, int N, int k1, int k2) {
    if (M <= 0 || N <= 0 || N % 8 != 0) return 1;
    return dense_plan(M, N, k1, k2, 8).splits;
}

int launch_dense(const GemmDesc& d, hipStream_t st) {
    if (d.M <= 0 || d.N <= 0) return QBLORA_OK;
    // whole 64-wide steps of 16-byte chunks, whole 32-row blocks
    if (d.out_f32 || d.C2 || d.C_lo || !d.W1 || d.K1 <= 0 || d.K1 % kBK != 0 || d.N % 32 != 0 ||
        (reinterpret_cast<uintptr_t>(d.W1) & 15))
        return QBLORA_ERR_UNSUPPORTED;
    const DensePlan p = dense_plan(d.M, d.N, d.K1, d.K2, d.splits > 1 ? 8 : 1);
    if (d.splits > 1 && p.splits != d.splits) return QBLORA_ERR_UNSUPPORTED;       // not what dense_splits said
    switch (p.shape) {
        case 0: return launch_cfg<4, 2>(d, st);
        // slices start far apart in both operands, and with a tile on every CU their copies take longer: 512 tokens of 4096 x
        // 11008 in four slices 203.6 us a call with two phases a step, 205.6 with one; unsliced calls 10 to 5 % the other way
        case 1: return d.splits > 1 ? launch_cfg<2, 2>(d, st) : launch_cfg<2, 2, true>(d, st);
        case 2: return launch_cfg<4, 1>(d, st);
        default: return launch_cfg<2, 1>(d, st);
    }
}

}  // namespace qblora
