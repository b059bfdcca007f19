// Dequantize-and-contract kernel of the adapted layer's forward for gfx950 (Alg. 1 qblora_forward:
// W_tilde = dequantize(...), x @ W_tilde, plus the adapter term), for calls whose scratch cannot hold the
// dequantized weight (few tokens; the forward that allocates nothing).
//
//   C[M,N] = X1[M,K1] * Wq^T  +  X2[M,K2] * W2[N/div2, K2]^T
//
// Segment 1 reads the 4-bit codes and block scales of the frozen base weight from HBM, rebuilds
// bf16 weights (Eq. 1: c[code]*alpha (+beta), fp32 then round-to-nearest-even) straight into an
// LDS tile and feeds them to v_mfma_f32_16x16x32_bf16 with fp32 accumulation; the dequantized
// weight never exists in HBM.  Segment 2 is a plain bf16 K-extension: the adapter's rank-R product
// rides in the same accumulators as R extra contraction steps (X2 = s*U, W2 = B^T with output row n using row
// n/lambda2, i.e. repeat_interleave).  k is accumulated in the order and by the instruction of dense.hip, so both
// give the same bits.
//
// Shape of the computation on a CU: one workgroup of 512 threads (8 wave64, two per SIMD) owns a
// 256 x 256 output tile; a wave owns 128 tokens x 64 features (128 accumulator registers).  Two waves per SIMD
// matter: the dequantization arithmetic of one wave issues in the shadow of the other wave's MFMAs.  Both operand
// tiles live in LDS as [row][64 k] bf16 (128 bytes per row) with the 16-byte chunks of a row XOR-swizzled by
// (row >> 1) & 7, double buffered, one barrier per k-step.  Activation tiles (and both bf16 tiles of segment 2)
// go from global memory directly into LDS (global_load_lds, 16 bytes per lane; the swizzle is applied by choosing
// which global chunk a lane fetches).  Codes and scales are fetched two k-steps ahead into registers and
// dequantized between the MFMAs of the step before they are needed, through a byte-indexed table
// in LDS that turns one byte of codes into two fp32 code values.
// The weight tile is the MFMA A operand and the token tile the B operand, so a lane ends up with 4
// consecutive output features of one token and stores them as one 8-byte word.
#include "common.h"

namespace qblora {

namespace {

constexpr int kThreads = 512;
constexpr int BM = 256, BN = 256, kBK = 64;
constexpr int kTileBytes = 256 * 128;                       // one operand tile: 256 rows x 128 bytes
constexpr int kTableBytes = 256 * 128;                      // byte-indexed pair table, 16 replicas

__device__ __align__(16) const uint32_t g_zero_chunk[4] = {0u, 0u, 0u, 0u};

__device__ __forceinline__ int swz(int row, int chunk) {
    return row * 128 + (((chunk ^ (row >> 1)) & 7) << 4);
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

// codes / scales of one k-step held in registers, 32 weights per thread: half a stored row (16 bytes of codes) and
// one scale -- or, with 8 x 8 quantization blocks (BR = 8), one scale per code dword (8 inputs = one block column)
template <int BR>
struct Staged {
    uint32_t cw[4];
    float sc[BR == 8 ? 4 : 1];
    float be[BR == 8 ? 4 : 1];
};

template <bool BETA, int BR>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_qlinear(GemmDesc d) {
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* sX = smem;                                   // 2 tiles
    unsigned char* sW = sX + 2 * kTileBytes;                    // 2 tiles
    unsigned char* sT = smem + 4 * kTileBytes;                  // pair table, see below

    // Every field of the descriptor the loop touches is copied into a local first: the copies in
    // the loop are assembly statements that clobber memory, and values must not be re-read around them.
    const int64_t M = d.M;
    const int N = d.N, d_in = d.d_in, K2 = d.K2, div2 = d.div2;
    const qblora_bf16* const X1 = d.X1; const int64_t ldx1 = d.ldx1;
    const qblora_bf16* const X2 = d.X2; const int64_t ldx2 = d.ldx2;
    const qblora_bf16* const W2 = d.W2; const int64_t ldw2 = d.ldw2;
    const uint8_t* const codes = d.codes;
    const float* const scales = d.scales;
    const float* const beta = d.beta;
    qblora_bf16* const C = reinterpret_cast<qblora_bf16*>(d.C);
    const int64_t ldc = d.ldc;
    const float out_scale = d.out_scale;

    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int wm0 = (wave & 1) * 128, wn0 = (wave >> 1) * 64;

    // ---- tile assignment: XCD-contiguous, grouped along tokens ---------------------------------
    const int tiles_m = (int)((M + BM - 1) / BM), tiles_n = (N + BN - 1) / BN;
    const int ntiles = tiles_m * tiles_n;
    int L = blockIdx.x;
    if ((ntiles & 7) == 0) L = (blockIdx.x & 7) * (ntiles >> 3) + (blockIdx.x >> 3);
    constexpr int GM = 4;
    const int in_group = GM * tiles_n;
    const int first_m = (L / in_group) * GM;
    const int gsize = min(tiles_m - first_m, GM);
    const int mt = first_m + (L % in_group) % gsize, nt = (L % in_group) / gsize;
    const int64_t m0 = (int64_t)mt * BM;
    const int n0 = nt * BN;

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
    }

    const int steps1 = d_in / kBK, steps2 = (K2 + kBK - 1) / kBK;
    const int nsteps = steps1 + steps2;
    const int bpr = d_in / kBlock;                // blocks per stored weight row

    f32x4 acc[4][8];                              // [16 features][16 tokens]
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 8; ++b) acc[a][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // ---- direct global -> LDS copies -------------------------------------------------------------
    // Wave w fills rows 32w .. 32w+31 of a tile with 4 copies of 8 rows each.  In copy i, lane l
    // lands on row 32w + 8i + (l>>3), physical chunk l&7, which must hold logical chunk
    // (l&7) ^ (row>>1)&7 = (l&7) ^ (4(i&1) + (l>>4)).
    const int crow = lane >> 3;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem) + wave * 32 * 128);
    // check_k: chunks at or beyond K are fetched from a zero constant instead (K-extension only)
    auto copy_tile = [&](const bool check_k, const qblora_bf16* src, int64_t ld, int64_t row_base, int64_t row_max,
                         int div, int K, int k0, uint32_t tile_off) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int64_t row = row_base + wave * 32 + i * 8 + crow;
            row = row > row_max ? row_max : row;
            if (div != 1) row = (int64_t)((uint32_t)row / (uint32_t)div);      // only weight rows (< 2^31) are divided
            const int k = k0 + (((lane & 7) ^ (4 * (i & 1) + (lane >> 4))) << 3);
            const qblora_bf16* p = src + row * ld + k;
            if (check_k)
                p = (k < K) ? p : reinterpret_cast<const qblora_bf16*>(g_zero_chunk);
            copy16_to_lds(p, lds0 + tile_off + i * 8 * 128);
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
    auto issue_x1 = [&](int step, int buf) __attribute__((always_inline)) {
        const qblora_bf16* base = x1_tile + step * kBK;
#pragma unroll
        for (int i = 0; i < 4; ++i) copy16_to_lds(base, xoff[i], lds0 + buf * kTileBytes + i * 8 * 128);
    };
    auto issue_copies = [&](int step, int buf) __attribute__((always_inline)) {
        if (step < steps1) {
            issue_x1(step, buf);
        } else {
            const int k0 = (step - steps1) * kBK;
            copy_tile(true, X2, ldx2, m0, M - 1, 1, K2, k0, buf * kTileBytes);
            copy_tile(true, W2, ldw2, n0, N - 1, div2, K2, k0, (2 + buf) * kTileBytes);
        }
    };

    // ---- codes / scales -> registers -------------------------------------------------------------
    const uint8_t* fwd_codes = nullptr; int fwd_stride = 32;
    const float* fwd_scales = nullptr; int fwd_scale_stride = 1;
    int qrow = n0 + (t >> 1);                        // this thread's stored weight row (it owns half of it)
    if (qrow > N - 1) qrow = N - 1;
    if (d.codes_tiled) { fwd_codes = d.codes_tiled + tiled_run_offset(n0 + (t >> 1), 0, bpr) + (t & 1) * 16; fwd_stride = 256 * 32; }
    else fwd_codes = codes + (int64_t)qrow * (d_in / 2) + (t & 1) * 16;
    if (d.scales_tiled) { fwd_scales = d.scales_tiled + tiled_run_offset(n0 + (t >> 1), 0, bpr) / 32; fwd_scale_stride = 256; }
    else fwd_scales = scales + (int64_t)qrow * bpr;
    auto load_staged = [&](Staged<BR>& s, int step) __attribute__((always_inline)) {
        const uint4 v = *reinterpret_cast<const uint4*>(fwd_codes + (int64_t)step * fwd_stride);
        s.cw[0] = v.x; s.cw[1] = v.y; s.cw[2] = v.z; s.cw[3] = v.w;
        if constexpr (BR == 8) {
            // block columns 8*step + 4*half .. +3 of block row qrow/8: one scale per code dword
            const int64_t b0 = (int64_t)(qrow >> 3) * (d_in >> 3) + 8 * step + 4 * (t & 1);
            const float4 a4 = *reinterpret_cast<const float4*>(scales + b0);
            s.sc[0] = a4.x; s.sc[1] = a4.y; s.sc[2] = a4.z; s.sc[3] = a4.w;
            if constexpr (BETA) {
                const float4 b4 = *reinterpret_cast<const float4*>(beta + b0);
                s.be[0] = b4.x; s.be[1] = b4.y; s.be[2] = b4.z; s.be[3] = b4.w;
            }
        } else {
            s.sc[0] = fwd_scales[(int64_t)step * fwd_scale_stride];
            if constexpr (BETA) s.be[0] = beta[(int64_t)qrow * bpr + step];
        }
    };

    // ---- dequantization of a staged k-step: 4 pieces of 8 weights (4 table reads each) per thread ----------
    // Piece p = code dword p of this thread's half row -> chunk 4*half+p of LDS row t>>1.
    constexpr int kPieces = 4, kReads = 4;
    const uint32_t table_lane = lds_address(sT) - lds_address(smem) + ((lane & 15) << 3);
    auto table_offsets = [&](const Staged<BR>& s, int p, uint32_t (&li)[kReads]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kReads; ++i) {           // byte i of dword p
            const uint32_t w = s.cw[p];
            const uint32_t sh = i == 0 ? (w << 7) : (w >> (8 * i - 7));
            li[i] = (sh & 0x7f80u) | table_lane;
        }
    };
    auto table_reads = [&](const uint32_t (&li)[kReads], float2 (&lv)[kReads]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kReads; ++i) lv[i] = *reinterpret_cast<const float2*>(smem + li[i]);
    };
    auto finish_piece = [&](const Staged<BR>& s, int p, const float2 (&lv)[kReads], unsigned char* tile)
        __attribute__((always_inline)) {
        float lo[kReads], hi[kReads];
#pragma unroll
        for (int i = 0; i < kReads; ++i) {
            const float sc = s.sc[BR == 8 ? p : 0], be = BETA ? s.be[BR == 8 ? p : 0] : 0.0f;
            lo[i] = BETA ? __fmaf_rn(lv[i].x, sc, be) : __fmul_rn(lv[i].x, sc);
            hi[i] = BETA ? __fmaf_rn(lv[i].y, sc, be) : __fmul_rn(lv[i].y, sc);
        }
        // byte i holds elements 2i, 2i+1 of the 8: adjacent k, packed as they come
        uint4 o0;
        o0.x = pack_bf16(lo[0], hi[0]); o0.y = pack_bf16(lo[1], hi[1]);
        o0.z = pack_bf16(lo[2], hi[2]); o0.w = pack_bf16(lo[3], hi[3]);
        *reinterpret_cast<uint4*>(tile + swz(t >> 1, 4 * (t & 1) + p)) = o0;
    };
    auto dequant_store = [&](const Staged<BR>& s, unsigned char* tile) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < kPieces; ++p) {
            uint32_t li[kReads];
            float2 lv[kReads];
            table_offsets(s, p, li);
            table_reads(li, lv);
            finish_piece(s, p, lv, tile);
        }
    };

    // ---- one k-step ----------------------------------------------------------------------------------
    // Four quarters of 16 MFMAs: a 32-wide slice of k, half of the wave's tokens.  Token fragments of quarter q+1
    // are read during quarter q (two sets), the slice's weight fragments at its start; the dequantization of the
    // next weight tile is spread over the first three quarters (table reads one quarter before the values are
    // scaled and stored); the barrier that publishes the next tiles sits in front of the last quarter, whose MFMAs
    // cover it and the first fragment reads of the next step.
    const int r = lane & 15, g = lane >> 4;
    bf16x8 wf[4], xf[2][4];         // token set 0 holds quarter 0 when a step starts
    // Fragment addresses: 16-row block b, slice ks: row base + 16b + r, chunk 4ks + g sits at (base + r)*128 +
    // 2048b + 16*[(g ^ r>>1) & 7 ^ 4ks] -- one per-lane value XOR a constant plus an immediate;
    // the empty asm in run_step keeps the variants from being hoisted and held in registers.
    uint32_t frag_w = (uint32_t)(sW - smem) + (uint32_t)((wn0 + r) * 128 + ((g ^ (r >> 1)) << 4));
    uint32_t frag_x = (uint32_t)(sX - smem) + (uint32_t)((wm0 + r) * 128 + ((g ^ (r >> 1)) << 4));
    auto read_x = [&](const unsigned char* bx, int q, bf16x8 (&fx)[4]) __attribute__((always_inline)) {
        const uint32_t xo = (uint32_t)(bx - sX);
#pragma unroll
        for (int b = 0; b < 4; ++b)
            fx[b] = *reinterpret_cast<const bf16x8*>(smem + ((frag_x ^ (uint32_t)((q >> 1) << 6)) + (xo + (4 * (q & 1) + b) * 2048)));
    };
    auto read_w = [&](const unsigned char* bw, int ks) __attribute__((always_inline)) {
        const uint32_t wo = (uint32_t)(bw - sW);
#pragma unroll
        for (int a = 0; a < 4; ++a) wf[a] = *reinterpret_cast<const bf16x8*>(smem + ((frag_w ^ (uint32_t)(ks << 6)) + (wo + a * 2048)));
    };
    // dq: dequantize `sdq` into bw_next during this step; has_next: a step follows (its tiles are in
    // bx_next / bw_next once the barrier is passed); dq_next: the following step dequantizes `sdq_next`, whose
    // first piece is looked up behind this step's barrier (lv0 carries the values across the step boundary).
    // All flags are literal `true` in the steady state.
    float2 lv0[kReads];
    auto run_step = [&](const unsigned char* bx, const unsigned char* bw, const unsigned char* bx_next,
                        unsigned char* bw_next, const bool dq, const Staged<BR>& sdq, const bool has_next,
                        const bool refill, const int step2, const int buf2, const bool dq_next,
                        const Staged<BR>& sdq_next) __attribute__((always_inline)) {
        float2 lv[2][kReads];
        uint32_t li[kReads];
        asm volatile("" : "+v"(frag_w), "+v"(frag_x));
        if (dq) {
#pragma unroll
            for (int i = 0; i < kReads; ++i) lv[0][i] = lv0[i];
        }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int cur = ks & 1, nxt = cur ^ 1;
            // the last piece is stored in front of the barrier that publishes the tile
            if (ks == 3 && dq) finish_piece(sdq, 3, lv[1], bw_next);
            if (ks == 3 && has_next) {
                __builtin_amdgcn_s_waitcnt(0x0F70);        // vmcnt(0): direct copies and staged codes
                __syncthreads();                           // next tiles published; this step's tiles free
                read_x(bx_next, 0, xf[0]);
                if (refill) issue_x1(step2, buf2);         // this step's token buffer is free: refill it
            }
            if (ks % 2 == 0) read_w(bw, ks / 2);
            if (ks < 3) read_x(bx, ks + 1, xf[nxt]);
            if (dq && ks < 3) {
                // piece ks+1 is looked up while piece ks is scaled and stored
                table_offsets(sdq, ks + 1, li);
                table_reads(li, lv[nxt]);
            }
            if (ks == 3 && dq_next) {                      // the staged codes of the next step's tile have arrived
                // (the empty statement pins the address arithmetic behind the barrier: hoisted to the top of
                // the step it would wait for the code loads issued there)
                Staged<BR> nx = sdq_next;
#pragma unroll
                for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(nx.cw[i]));
                table_offsets(nx, 0, li);
                table_reads(li, lv0);
            }
            __builtin_amdgcn_sched_barrier(0);             // LDS reads of the next quarter go out before this quarter's MFMAs
            if (dq && ks < 3) finish_piece(sdq, ks, lv[cur], bw_next);
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    acc[a][4 * (ks & 1) + b] =
                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[a], xf[cur][b], acc[a][4 * (ks & 1) + b], 0, 0, 0);
            // the scaling arithmetic of the piece goes into the shadow of the MFMAs, one vector instruction each
#pragma unroll
            for (int i = 0; i < 15; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 1, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // ---- main loop ---------------------------------------------------------------------------------
    // Invariant at the top of step s: tile buffers s&1 hold step s and fragment set 0 holds its first
    // quarter; st[(s+1)&1] holds the codes of step s+1 (if that is a quantized step).
    Staged<BR> st[2];
    if (nsteps > 0) {
        issue_copies(0, 0);
        int issued = 0;                                    // copies are in flight or done for steps <= issued
        if (steps1 > 1) { issue_copies(1, 1); issued = 1; }
        if (steps1 > 0) load_staged(st[0], 0);
        if (steps1 > 1) load_staged(st[1], 1);
        __syncthreads();                                   // pair table visible
        if (steps1 > 0) dequant_store(st[0], sW);
        __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();
        read_x(sX, 0, xf[0]);
        if (steps1 > 1) {                                  // first piece of the tile the first step dequantizes
            uint32_t li[kReads];
            table_offsets(st[1], 0, li);
            table_reads(li, lv0);
        }
        int s = 0;
        // Quantized steps whose successor is quantized too (the successor's tile is dequantized during
        // the step), unrolled by two so that the staging registers and the tile buffers have fixed
        // names.  Codes are fetched two steps ahead; past the end the last quantized step is fetched
        // again (in bounds, unused) so that the body has no conditions.  A step refills its own token
        // buffer with the copies of the step after next (when that is a quantized step) behind its
        // barrier, under its last 8 MFMAs.
        const int last_q = steps1 - 1;
        for (; s + 2 < steps1; s += 2) {
            load_staged(st[0], min(s + 2, last_q));
            run_step(sX, sW, sX + kTileBytes, sW + kTileBytes, true, st[1], true, true, s + 2, 0, true, st[0]);
            load_staged(st[1], min(s + 3, last_q));
            const bool more = s + 3 < steps1;
            // (past the last dequantizing step the looked-up piece is simply not used)
            run_step(sX + kTileBytes, sW + kTileBytes, sX, sW, true, st[0], true, more, s + 3, 1, true, st[1]);
            issued = more ? s + 3 : s + 2;
        }
        if (s + 1 < steps1) {
            run_step(sX, sW, sX + kTileBytes, sW + kTileBytes, true, st[1], true, false, 0, 0, false, st[0]);
            ++s;
        }
        // the last quantized step and the K-extension steps: nothing to dequantize; copies of the next
        // step are issued at the top of a step when no earlier step has done it
        for (; s < nsteps; ++s) {
            const int buf = s & 1;
            const bool has_next = s + 1 < nsteps;
            if (has_next && issued < s + 1) { issue_copies(s + 1, buf ^ 1); issued = s + 1; }
            run_step(sX + buf * kTileBytes, sW + buf * kTileBytes, sX + (buf ^ 1) * kTileBytes,
                     sW + (buf ^ 1) * kTileBytes, false, st[0], has_next, false, 0, 0, false, st[0]);
        }
    }

    __builtin_amdgcn_s_waitcnt(0x0F70);                    // nothing may still be writing this workgroup's LDS

    // ---- epilogue ---------------------------------------------------------------------------------------
    // A lane holds features n..n+3 of one token per accumulator, i.e. 8 bytes of an output row.
    // The wave first lays its 128 x 64 quadrant out in LDS (the tiles are dead by now) as bf16 rows of
    // 128 bytes (pitch 144), then reads it back 16 bytes per lane so that every global store
    // instruction writes eight complete 128-byte row segments.
    __syncthreads();                                       // every wave is done reading the tiles
    {
        constexpr int kPitch = 144;
        unsigned char* eb = smem + wave * (128 * kPitch);
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                uint2 o;
                o.x = pack_bf16(acc[a][b][0] * out_scale, acc[a][b][1] * out_scale);
                o.y = pack_bf16(acc[a][b][2] * out_scale, acc[a][b][3] * out_scale);
                *reinterpret_cast<uint2*>(eb + (b * 16 + r) * kPitch + (a * 16 + g * 4) * 2) = o;
            }
        const int erow = lane >> 3, echunk = lane & 7;
        const int n = n0 + wn0 + echunk * 8;
#pragma unroll 8
        for (int i = 0; i < 16; ++i) {
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

template <bool BETA, int BR>
int launch_cfg(const GemmDesc& d, hipStream_t st) {
    constexpr size_t smem = 4 * kTileBytes + kTableBytes;
    auto kern = k_qlinear<BETA, BR>;
    // set once per instantiation; the initialisation of a function-local static is thread safe
    static const bool attr_ok = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem) == hipSuccess;
    if (!attr_ok) return QBLORA_ERR_LAUNCH;
    int64_t tiles = ((d.M + BM - 1) / BM) * ((d.N + BN - 1) / BN);
    hipLaunchKernelGGL(kern, dim3((unsigned)tiles), dim3(kThreads), smem, st, d);
    return launch_status();
}

}  // namespace

// The quantized GEMM of the layer's forward (qmode 1, bf16 output, no auxiliary outputs).
int launch_qlinear(const GemmDesc& d, hipStream_t st) {
    if (d.M <= 0 || d.N <= 0) return QBLORA_OK;
    if (d.out_f32 || d.C2 || d.C_lo) return QBLORA_ERR_UNSUPPORTED;
    if (d.block_rows == 8) {
        // scales / offsets are read as 16-byte groups of 4 block columns; tile-ordered scales do not exist
        if (d.scales_tiled || !d.scales || d.d_out % 8 != 0 || (reinterpret_cast<uintptr_t>(d.scales) & 15) ||
            (reinterpret_cast<uintptr_t>(d.beta) & 15))
            return QBLORA_ERR_UNSUPPORTED;
        return d.beta ? launch_cfg<true, 8>(d, st) : launch_cfg<false, 8>(d, st);
    }
    return d.beta ? launch_cfg<true, 1>(d, st) : launch_cfg<false, 1>(d, st);
}

}  // namespace qblora
