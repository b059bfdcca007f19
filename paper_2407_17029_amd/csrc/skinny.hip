// Narrow-output bf16 GEMM of the adapter path for gfx950:
//
//   C[M,N] = out_scale * X[M,K] * W[N,K]^T,   N = the adapter's inner rank R (tens to a few hundred)
//
// used for U = P A (Sec. 3.2; the average pool is folded into W = A^T repeated lambda1 times along
// k, so X is the raw activation) and for dU = dV B^T of the backward pass (the sum pool over lambda2
// folded the same way).  M is the token count and K the layer width, so the kernel reads X once
// from HBM and is bound by that stream, not by the MFMAs: the design goal is bytes in flight.
//
// One workgroup of 4 wave64 owns BM tokens x BN output columns and walks K through a ring of LDS
// stages (one or two 64-wide k-steps per stage and barrier).  Both operand tiles of a stage arrive by
// direct global -> LDS copies issued STAGES-1 stages ahead.  X comes from HBM once; W (1 MB for rank
// 128 at K = 4096) is re-read from L2 by every token tile, so the traffic through the CUs is a few
// times the X stream and that, not HBM latency, sets the pace: measured times do not change between
// 3 and 9 stages.  With a token count that gives only 128 tiles of 64 tokens, 64 x 64 tiles put a
// workgroup on every CU; the two workgroups that share a token tile sit on the same XCD and the second
// finds X in L2.  Tiles are [row][64 k] bf16 with the 16-byte chunks XOR-swizzled by
// (row ^ row>>3) & 7, applied by choosing which global chunk a lane fetches.
//
// Few tokens leave most of the chip idle (512 tokens x 128 columns: 16 workgroups) while each workgroup is a serial
// chain of barriers and LDS round trips (1000 cycles per 128 k, the matrix pipe busy for a quarter of them).  The
// contraction is then cut into slices, one workgroup each, whose fp32 partial tiles k_skinny_reduce adds in slice
// order.
//
// W is read where it lies wherever the pool / repeat factor is 1 or 2: B as rows of k, A the other way round, one row per
// stored k.  A's tile is turned by the transposing LDS read (ds_read_b64_tr_b16, see grads.hip), so that the kernel waits for no
// copy of A and the re-layouts that others wait for share its launch.  Any K of whole 64-wide steps goes through the two-step
// stages; the last may be half full.  us a call (forward and backward) with a copy of A in a launch of its own and slices only
// where K is whole stages / now: 512 tokens of 11008 x 4096, rank 64, 212.8 / 204.1; 1337 of 5120 x 5120 221.5 / 213.0; 334 of
// 4224 x 8000 193.8 / 167.8 (K = 8000 unsliced 33 us); 154 of 14016 x 896 at lambda 8, whose copies are half as wide, 201.8 / 146.3.
#include <algorithm>

#include "dequant.h"
#include "prep.h"

namespace qblora {

namespace {

constexpr int kThreads = 256;
constexpr int kBK = 64;

// s_waitcnt immediate that waits until at most n vector-memory operations are outstanding
constexpr int vmcnt_imm(int n) { return (n & 15) | 0x0F70 | ((n >> 4) << 14); }

__device__ __forceinline__ int swz(int row, int chunk) {
    return row * 128 + (((chunk ^ row ^ (row >> 3)) & 7) << 4);
}

__device__ __forceinline__ void copy16_to_lds(const void* uniform_base, uint32_t lane_offset, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_base), "v"(lane_offset), "s"(uniform_base) : "memory");
}

__device__ __forceinline__ uint32_t lds_address(const void* p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

typedef __attribute__((ext_vector_type(4))) short s16x4;
__device__ __forceinline__ uint2 tr_read(const unsigned char* p) {
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p)));
}

// kDup = 2: W is stored with K/2 columns and column m serves k = 2m and 2m+1 (the adapter operand
// before its expansion along k: the pool over pairs of features is then folded into the fragment,
// which halves the W stream from L2 and its LDS tile).  Only in the k-split form with two k-steps per
// stage: the W columns of both k-steps are 128 contiguous bytes per row and form one tile per stage,
// behind the stage's two X sub-tiles.
// kByK: W is stored [K/kDup][N].  The tile of a stage is its 128/kDup rows of BN columns, behind the X sub-tiles as well, with the
// 16-byte chunks of a row swizzled by (row >> 1 & 1) << 2 (64 columns) or (row & 3) << 2 (128), so that the four rows of a
// transposing read lie in different banks.
template <int BM, int BN, int kStages, int kSub, bool kSplitK, int kDup, bool kByK>
__device__ __forceinline__ void skinny_tile(const GemmDesc& d, const unsigned block, unsigned char* const smem) {
    static_assert(!kSplitK || (BM == 64 && (BN == 64 || BN == 128)), "the k-split form is written for 64 x 64 and 64 x 128 tiles");
    static_assert((kDup == 1 && !kByK) || (kDup <= 2 && kSplitK && kSub == 2), "W unexpanded: k-split form, two k-steps per stage");
    // a stage holds kSub consecutive k-steps (sub-tiles of 64 k each): one barrier per kSub * 64 k
    constexpr int kXBytes = BM * 128, kWBytes = BN * 128 / kDup, kSubBytes = kXBytes + kWBytes, kStageBytes = kSub * kSubBytes;
    constexpr bool kOneW = kDup == 2 || kByK;     // one W tile per stage
    constexpr int XC = BM / 32, WC = kOneW ? kSub * kWBytes / 4096 : BN / 32;     // copies per wave and sub-tile (kOneW: W copies per stage)
    // byte offsets of the X sub-tile u and of its W tile inside a stage
    auto x_at = [](int u) { return kOneW ? u * kXBytes : u * kSubBytes; };
    auto w_at = [](int u) { return kOneW ? kSub * kXBytes : u * kSubBytes + kXBytes; };
    constexpr int WN = BN / 32, WM = 4 / WN;      // waves along the columns / along the tokens
    constexpr int MF = BM / (32 * WM);            // 32-token blocks per wave
    static_assert(MF >= 1 && WN * WM == 4, "tile shape");
    const int64_t M = d.M;
    const int N = d.N, K = d.K2;
    const qblora_bf16* const X = d.X2; const int64_t ldx = d.ldx2;
    const qblora_bf16* const W = d.W2; const int64_t ldw = d.ldw2;
    qblora_bf16* const C = reinterpret_cast<qblora_bf16*>(d.C);
    qblora_bf16* const C2 = d.C2;
    qblora_bf16* const C_lo = d.C_lo;
    const int64_t ldc = d.ldc;
    const float out_scale = d.out_scale, c2_scale = d.c2_scale;

    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    // blockIdx.x % 8 is the XCD: the column tiles of one token tile are 8 apart
    const int tiles_n = (N + BN - 1) / BN;
    const int splits = d.splits > 1 ? d.splits : 1, all_steps = (K / kBK + kSub - 1) / kSub;
    int z = 0, bid = block, step0 = 0, nsteps = all_steps;    // (unsliced calls spend no divisions on it: 0.3 us)
    if (splits > 1) {
        z = bid % splits; bid /= splits;
        step0 = all_steps * z / splits;           // all_steps < 2^24
        nsteps = all_steps * (z + 1) / splits - step0;             // at least one: splits <= all_steps
    }
    const int nsub = K / kBK - step0 * kSub;      // 64-wide steps from here on: the last stage of all may hold one
    const int grp = bid / (8 * tiles_n), within = bid % (8 * tiles_n);
    const int64_t m0 = ((int64_t)grp * 8 + (within & 7)) * BM;
    const int n0 = (within >> 3) * BN;
    if (m0 >= M) return;                          // the grid is rounded up to whole groups of 8 token tiles
    const int wave_n = wave % WN, wave_m = wave / WN;

    // per-lane byte offsets of the copies, relative to the first row of the tile
    const int crow = lane >> 3;
    uint32_t xoff[XC], woff[WC];
#pragma unroll
    for (int i = 0; i < XC; ++i) {
        int64_t lrow = wave * (8 * XC) + i * 8 + crow;
        if (m0 + lrow > M - 1) lrow = M - 1 - m0;
        xoff[i] = (uint32_t)(lrow * ldx * 2) + (((lane & 7) ^ crow ^ ((XC * wave + i) & 7)) << 4);
    }
    // by k: RPI rows of CPR chunks a copy; columns past N read the last chunk of the row and are never stored
    constexpr int CPR = BN / 8, RPI = 64 / CPR;
    const int kchunk = min(n0 / 8 + ((lane % CPR) ^ ((BN == 64 ? (lane / CPR) >> 1 & 1 : (lane / CPR) & 3) << 2)), (N >> 3) - 1);
    const int wchunk = (lane & 7) ^ crow;         // by row: ^ the copy's number
#pragma unroll
    for (int i = 0; i < WC; ++i) {
        if constexpr (kByK) {
            const int krow = (wave * WC + i) * RPI + lane / CPR;
            woff[i] = (uint32_t)((int64_t)krow * ldw * 2) + (uint32_t)(kchunk << 4);
        } else {
            int lrow = wave * (8 * WC) + i * 8 + crow;
            if (n0 + lrow > N - 1) lrow = N - 1 - n0;
            woff[i] = (uint32_t)((int64_t)lrow * ldw * 2) + ((wchunk ^ ((WC * wave + i) & 7)) << 4);
        }
    }
    const qblora_bf16* const x_tile = X + m0 * ldx + (int64_t)step0 * kSub * kBK;
    const qblora_bf16* const w_tile = kByK ? W + (int64_t)step0 * kSub * (kBK / kDup) * ldw
                                           : W + (int64_t)n0 * ldw + (int64_t)step0 * kSub * (kBK / kDup);
    const uint32_t lds_x = __builtin_amdgcn_readfirstlane(lds_address(smem) + wave * (8 * XC) * 128);
    const uint32_t lds_w = __builtin_amdgcn_readfirstlane(lds_address(smem) + wave * WC * 1024);
    auto issue = [&](int step) __attribute__((always_inline)) {
        const uint32_t stage = (step % kStages) * kStageBytes;
#pragma unroll
        for (int u = 0; u < kSub; ++u) {
            if (u > 0 && step * kSub + u >= nsub) break;                  // fewer copies: only in the very last stage
            const qblora_bf16* xb = x_tile + (step * kSub + u) * kBK;
#pragma unroll
            for (int i = 0; i < XC; ++i) copy16_to_lds(xb, xoff[i], lds_x + stage + x_at(u) + i * 8 * 128);
            if (kOneW && u > 0) continue;         // one W tile per stage: stored columns (rows) of both k-steps
            const qblora_bf16* wb = w_tile + (int64_t)(step * kSub + u) * (kBK / kDup) * (kByK ? ldw : 1);
            const bool half = kOneW && step * kSub + 1 >= nsub;           // the second half of the tile does not exist
#pragma unroll
            for (int i = 0; i < WC; ++i) {
                uint32_t off = woff[i];
                if (half) {                                               // ... its lanes fetch the first half again
                    if constexpr (kByK) off -= (wave * WC + i) * RPI + lane / CPR >= kBK / kDup ? (uint32_t)((kBK / kDup) * ldw * 2) : 0u;
                    else off -= (wchunk ^ ((WC * wave + i) & 7)) & 4 ? 64u : 0u;
                }
                copy16_to_lds(wb, off, lds_w + stage + w_at(u) + i * 1024);
            }
        }
    };

    // Plain form: a wave owns 32 columns x MF token blocks and keeps one accumulator chain per
    // sub-tile (added at the end).  k-split form (64 tokens x 64 or 128 columns): a 32 x 32 wave tile would
    // read two fragments per MFMA, which is all the LDS can deliver; instead every wave computes the whole
    // tile (acc[column block][token block]) for one quarter of each sub-tile's k (slice ks == wave), one
    // fragment read per MFMA (three per four with 128 columns), and the four partial tiles are added through
    // LDS at the end, 64 columns at a time.
    constexpr int NA = kSplitK ? BN / 32 : kSub, NB = kSplitK ? 2 : MF;
    f32x16 acc[NA][NB];
#pragma unroll
    for (int u = 0; u < NA; ++u)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[u][b][i] = 0.0f;

    const int r = lane & 31, hi = lane >> 5;
    // by k: lane s of a group of 16 points at row s >> 2, columns 4*(s & 3) .. +3 of the group's 16, and receives column s
    uint32_t kfrag = 0;
    if constexpr (kByK) {
        const int srow = hi * 8 / kDup + ((lane & 15) >> 2), col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
        kfrag = (uint32_t)(srow * BN * 2 + (((col >> 3) ^ ((BN == 64 ? (srow >> 1) & 1 : srow & 3) << 2)) << 4) + (col & 4) * 2);
    }
    auto compute = [&](int step) __attribute__((always_inline)) {
        if constexpr (kSplitK) {
#pragma unroll
            for (int u = 0; u < kSub; ++u) {
                if (u > 0 && step * kSub + u >= nsub) break;
                const unsigned char* bx = smem + (step % kStages) * kStageBytes + x_at(u);
                const unsigned char* bw = smem + (step % kStages) * kStageBytes + w_at(u);
                bf16x8 wf[NA], xf[2];
#pragma unroll
                for (int a = 0; a < 2; ++a) xf[a] = *reinterpret_cast<const bf16x8*>(bx + swz(a * 32 + r, wave * 2 + hi));
#pragma unroll
                for (int a = 0; a < NA; ++a) {
                    if constexpr (kByK) {
                        // stored rows of k = 64*u + 16*wave + 8*hi .. +7, columns a*32 + r
                        const unsigned char* const p = bw + ((u * kBK + wave * 16) / kDup) * (BN * 2) + (kfrag ^ (uint32_t)(a << 6));
                        const uint2 v = tr_read(p);
                        uint4 e;
                        if constexpr (kDup == 2) {
                            e = make_uint4(__builtin_amdgcn_perm(v.x, v.x, 0x01000100u), __builtin_amdgcn_perm(v.x, v.x, 0x03020302u),
                                           __builtin_amdgcn_perm(v.y, v.y, 0x01000100u), __builtin_amdgcn_perm(v.y, v.y, 0x03020302u));
                        } else {
                            const uint2 w = tr_read(p + 4 * BN * 2);
                            e = make_uint4(v.x, v.y, w.x, w.y);
                        }
                        wf[a] = __builtin_bit_cast(bf16x8, e);
                    } else if constexpr (kDup == 2) {
                        // stored columns 32*u + 8*wave + 4*hi .. +3 of row a*32 + r, each used for two k
                        const uint2 v = *reinterpret_cast<const uint2*>(bw + swz(a * 32 + r, 4 * u + wave) + 8 * hi);
                        const uint4 e = make_uint4(__builtin_amdgcn_perm(v.x, v.x, 0x01000100u), __builtin_amdgcn_perm(v.x, v.x, 0x03020302u),
                                                   __builtin_amdgcn_perm(v.y, v.y, 0x01000100u), __builtin_amdgcn_perm(v.y, v.y, 0x03020302u));
                        wf[a] = __builtin_bit_cast(bf16x8, e);
                    } else {
                        wf[a] = *reinterpret_cast<const bf16x8*>(bw + swz(a * 32 + r, wave * 2 + hi));
                    }
                }
#pragma unroll
                for (int a = 0; a < NA; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[a], xf[b], acc[a][b], 0, 0, 0);
            }
            return;
        }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int u = 0; u < kSub; ++u) {
                const unsigned char* bx = smem + (step % kStages) * kStageBytes + x_at(u);
                const unsigned char* bw = smem + (step % kStages) * kStageBytes + w_at(u);
                const bf16x8 wf = *reinterpret_cast<const bf16x8*>(bw + swz(wave_n * 32 + r, ks * 2 + hi));
#pragma unroll
                for (int b = 0; b < MF; ++b) {
                    const bf16x8 xf = *reinterpret_cast<const bf16x8*>(bx + swz((wave_m * MF + b) * 32 + r, ks * 2 + hi));
                    acc[u][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, xf, acc[u][b], 0, 0, 0);
                }
            }
    };

    constexpr int kAhead = kStages - 1;           // stages in flight
#pragma unroll
    for (int i = 0; i < kAhead; ++i)
        if (i < nsteps) issue(i);
    int s = 0;
    for (; s + kAhead < nsteps; ++s) {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((kAhead - 1) * (XC * kSub + WC * (kOneW ? 1 : kSub))));   // the younger stages may be in flight
        __syncthreads();                          // stage s landed for all; everyone is done with step s-1
        issue(s + kAhead);                        // into the buffer step s-1 used
        compute(s);
    }
    for (; s < nsteps; ++s) {
        __builtin_amdgcn_s_waitcnt(0x0F70);       // vmcnt(0)
        __syncthreads();
        compute(s);
    }

    // lane holds columns n..n+3 of one token per accumulator quad of a 32 x 32 block
    auto emit = [&](const f32x16& v, const int out_n, const int out_m) __attribute__((always_inline)) {
        const int64_t m = m0 + out_m + r;
        if (m >= M) return;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int n = n0 + out_n + q * 8 + hi * 4;
            if (n >= N) continue;
            if (splits > 1) {                     // N % 4 == 0: whole 16-byte words
                *reinterpret_cast<float4*>(d.part + ((int64_t)z * M + m) * N + n) =
                    make_float4(v[q * 4 + 0], v[q * 4 + 1], v[q * 4 + 2], v[q * 4 + 3]);
                continue;
            }
            const float v0 = v[q * 4 + 0] * out_scale, v1 = v[q * 4 + 1] * out_scale;
            const float v2 = v[q * 4 + 2] * out_scale, v3 = v[q * 4 + 3] * out_scale;
            uint2 h;
            h.x = pack_bf16(v0, v1); h.y = pack_bf16(v2, v3);
            *reinterpret_cast<uint2*>(C + m * ldc + n) = h;
            if (C_lo) {
                uint2 o;
                o.x = pack_bf16(v0 - bf16_bits_to_float(h.x & 0xffffu), v1 - bf16_bits_to_float(h.x >> 16));
                o.y = pack_bf16(v2 - bf16_bits_to_float(h.y & 0xffffu), v3 - bf16_bits_to_float(h.y >> 16));
                *reinterpret_cast<uint2*>(C_lo + m * ldc + n) = o;
            }
            if (C2) {
                uint2 o;
                o.x = pack_bf16(v0 * c2_scale, v1 * c2_scale);
                o.y = pack_bf16(v2 * c2_scale, v3 * c2_scale);
                *reinterpret_cast<uint2*>(C2 + m * ldc + n) = o;
            }
        }
    };
    if constexpr (kSplitK) {
        // partial tiles -> LDS, 64 columns (two column blocks) per pass: register i of block (a, b) of wave w at
        // float [((w*4 + a*2+b)*16 + i)*64 + lane]; wave w then adds the four partials of block (a, b) =
        // (w >> 1, w & 1) in wave order.  The first barrier also ends the last step's reads of the ring.
        float* red = reinterpret_cast<float*>(smem);
#pragma unroll
        for (int p = 0; p < NA / 2; ++p) {
            __syncthreads();
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int i = 0; i < 16; ++i) red[((wave * 4 + a * 2 + b) * 16 + i) * 64 + lane] = acc[2 * p + a][b][i];
            __syncthreads();
            f32x16 sum;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                float v = red[((0 * 4 + wave) * 16 + i) * 64 + lane];
#pragma unroll
                for (int w = 1; w < 4; ++w) v += red[((w * 4 + wave) * 16 + i) * 64 + lane];
                sum[i] = v;
            }
            emit(sum, p * 64 + (wave >> 1) * 32, (wave & 1) * 32);
        }
    } else {
#pragma unroll
        for (int u = 1; u < kSub; ++u)
#pragma unroll
            for (int b = 0; b < MF; ++b)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[0][b][i] += acc[u][b][i];
#pragma unroll
        for (int b = 0; b < MF; ++b) emit(acc[0][b], wave_n * 32, (wave_m * MF + b) * 32);
    }
}

// One GEMM; or two that do not depend on each other (a backward that recomputes s*U beside dU), the first n_a workgroups on
// `a`, whose W is stored by row; or one and re-layouts that it does not wait for.  All compile-time: the choice costs a lone
// GEMM 0.5 us of scalar loads before its first copy.
struct SkinnyPair { GemmDesc a, b; unsigned n_a; };
struct SkinnyPrep { GemmDesc a; PrepDesc prep; unsigned n_a; };

template <int BM, int BN, int kStages, int kSub, bool kSplitK, int kDup, bool kByK>
__global__ __launch_bounds__(kThreads) void k_skinny(GemmDesc d) {
    extern __shared__ __align__(16) unsigned char smem[];
    skinny_tile<BM, BN, kStages, kSub, kSplitK, kDup, kByK>(d, blockIdx.x, smem);
}
template <int BM, int BN, int kStages, int kSub, bool kSplitK, int kDup, bool kByK>
__global__ __launch_bounds__(kThreads) void k_skinny_pair(SkinnyPair p) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (blockIdx.x < p.n_a) skinny_tile<BM, BN, kStages, kSub, kSplitK, kDup, false>(p.a, blockIdx.x, smem);
    else skinny_tile<BM, BN, kStages, kSub, kSplitK, kDup, kByK>(p.b, blockIdx.x - p.n_a, smem);
}
template <int BM, int BN, int kStages, int kSub, bool kSplitK, int kDup, bool kByK>
__global__ __launch_bounds__(kThreads) void k_skinny_prep(SkinnyPrep p) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (blockIdx.x < p.n_a) skinny_tile<BM, BN, kStages, kSub, kSplitK, kDup, kByK>(p.a, blockIdx.x, smem);
    else prep_block(p.prep, (int)(blockIdx.x - p.n_a), smem);
}

// The slices' partial tiles added in slice order, four columns of one token per thread; the same outputs as the
// unsplit kernel's epilogue.
__device__ __forceinline__ void skinny_sum(const GemmDesc& d, const unsigned block) {
    const int64_t i = ((int64_t)block * 256 + threadIdx.x) * 4, plane = d.M * d.N;
    if (i >= plane) return;
    float4 sum = *reinterpret_cast<const float4*>(d.part + i);
    for (int z0 = 1; z0 < d.splits; z0 += 8) {
        float4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const float4*>(d.part + min(z0 + u, d.splits - 1) * plane + i);
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (z0 + u < d.splits) { sum.x += v[u].x; sum.y += v[u].y; sum.z += v[u].z; sum.w += v[u].w; }
    }
    const int64_t m = i / d.N, o = m * d.ldc + (i - m * d.N);
    const float v0 = sum.x * d.out_scale, v1 = sum.y * d.out_scale, v2 = sum.z * d.out_scale, v3 = sum.w * d.out_scale;
    const uint2 h = make_uint2(pack_bf16(v0, v1), pack_bf16(v2, v3));
    *reinterpret_cast<uint2*>(reinterpret_cast<qblora_bf16*>(d.C) + o) = h;
    if (d.C_lo)
        *reinterpret_cast<uint2*>(d.C_lo + o) =
            make_uint2(pack_bf16(v0 - bf16_bits_to_float(h.x & 0xffffu), v1 - bf16_bits_to_float(h.x >> 16)),
                       pack_bf16(v2 - bf16_bits_to_float(h.y & 0xffffu), v3 - bf16_bits_to_float(h.y >> 16)));
    if (d.C2)
        *reinterpret_cast<uint2*>(d.C2 + o) =
            make_uint2(pack_bf16(v0 * d.c2_scale, v1 * d.c2_scale), pack_bf16(v2 * d.c2_scale, v3 * d.c2_scale));
}

template <bool kPair>
__global__ __launch_bounds__(256) void k_skinny_reduce(SkinnyPair p) {
    if (!kPair || blockIdx.x < p.n_a) skinny_sum(p.a, blockIdx.x);
    else skinny_sum(p.b, blockIdx.x - p.n_a);
}
// ... and behind them the weight of a call that dequantizes it once: the sums wait on a few cache lines while it streams.
template <bool BETA, int GEOM>
__global__ __launch_bounds__(256) void k_skinny_reduce_dequantize(GemmDesc d, unsigned n, DequantDesc q) {
    __shared__ __align__(16) DequantLds lds;
    if (blockIdx.x < n) skinny_sum(d, blockIdx.x);
    else dequantize_block<BETA, GEOM>(q, blockIdx.x - n, lds);
}

}  // namespace

// Whether the narrow GEMM can take W unexpanded: the k-split form with two k-steps per stage handles it (at every token
// count: with 512 or more tiles of 64 x 128 the plain form on the expanded operand measured slower, 13B layer at rank 128
// 21.0 -> 20.8 ms).  ldw: of W stored by row.
bool skinny_dup_applies(int N, int K, int64_t ldw) {
    return N >= 8 && N % 4 == 0 && N <= 512 && K % kBK == 0 && ldw % 8 == 0;
}

// Whether launch_skinny can take this problem (otherwise the general tile kernel does).
bool skinny_applies(const GemmDesc& d) {
    return d.qmode == 0 && !d.out_f32 && d.div2 == 1 && d.N % 4 == 0 && d.N <= 512 && d.K2 > 0 &&
           d.K2 % kBK == 0 && d.M >= 1 && (int64_t)128 * d.ldw2 * 2 < (int64_t)1 << 31 &&
           (int64_t)64 * d.ldx2 * 2 < (int64_t)1 << 31 && (!d.by_k || (d.N % 8 == 0 && d.ldw2 % 8 == 0));
}

namespace {

struct Call { const GemmDesc& d; const GemmDesc* b; const PrepDesc* prep; const DequantDesc* weight; };

// set once per kernel; callers keep the result in a function-local static, whose initialisation is thread safe
template <typename K>
bool set_lds(K kernel, size_t smem) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)smem) == hipSuccess;
}

template <int BM, int BN, int kStages, int kSub, bool kSplitK, int kDup = 1, bool kByK = false>
int launch_cfg(const Call& c, hipStream_t st) {
    constexpr size_t smem = kStages * kSub * (BM * 128 + BN * 128 / kDup);
    const GemmDesc& d = c.d;
    auto blocks = [](const GemmDesc& g) {
        const int64_t tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
        return (unsigned)((tiles_m + 7) / 8 * 8 * tiles_n * (kSplitK && g.splits > 1 ? g.splits : 1));
    };
    const unsigned n = blocks(d);
    if (c.b) {
        auto kern = k_skinny_pair<BM, BN, kStages, kSub, kSplitK, kDup, kByK>;
        static const bool ok = set_lds(kern, smem);
        if (!ok) return QBLORA_ERR_LAUNCH;
        hipLaunchKernelGGL(kern, dim3(n + blocks(*c.b)), dim3(kThreads), smem, st, SkinnyPair{d, *c.b, n});
    } else if (c.prep && kByK) {
        if constexpr (kByK) {
            static_assert(smem >= (size_t)kPrepLds, "both jobs share the LDS");
            auto kern = k_skinny_prep<BM, BN, kStages, kSub, kSplitK, kDup, kByK>;
            static const bool ok = set_lds(kern, smem);
            if (!ok) return QBLORA_ERR_LAUNCH;
            ProfileScope ev(QBLORA_PROFILE_PREP, st);
            hipLaunchKernelGGL(kern, dim3(n + (unsigned)c.prep->blocks()), dim3(kThreads), smem, st, SkinnyPrep{d, *c.prep, n});
        }
    } else {
        auto kern = k_skinny<BM, BN, kStages, kSub, kSplitK, kDup, kByK>;
        static const bool ok = set_lds(kern, smem);
        if (!ok) return QBLORA_ERR_LAUNCH;
        hipLaunchKernelGGL(kern, dim3(n), dim3(kThreads), smem, st, d);
    }
    if (kSplitK && d.splits > 1) {
        auto sums = [](const GemmDesc& g) { return (unsigned)((g.M * g.N / 4 + 255) / 256); };
        const unsigned m = sums(d);
        if (c.b) hipLaunchKernelGGL(k_skinny_reduce<true>, dim3(m + sums(*c.b)), dim3(256), 0, st, SkinnyPair{d, *c.b, m});
        else if (c.weight) {
            ProfileScope ev(QBLORA_PROFILE_DEQUANT, st);
            with_form(*c.weight, [&](auto beta, auto geom) {
                hipLaunchKernelGGL((k_skinny_reduce_dequantize<beta.value, geom.value>), dim3(m + c.weight->blocks), dim3(256), 0, st, d, m, *c.weight);
            });
        } else hipLaunchKernelGGL(k_skinny_reduce<false>, dim3(m), dim3(256), 0, st, SkinnyPair{d, d, m});
    }
    return launch_status();
}

}  // namespace

// A slice keeps at least four steps of 128 k (prologue and epilogue cost about five), and the split has to save twelve
// steps of about 0.44 us to pay for the second launch (4-5 us).  512 tokens, 128 columns: K = 4096 14.2 -> 5.5 + 4.6 us
// in 8 slices, K = 11008 32.5 -> 6.8 + 4.6 us in 16; 1337 tokens, 64 columns, K = 5120: 22 -> 6.8 + 4.2 us in 10.
int skinny_splits(int64_t M, int N, int K, int64_t max_part_bytes) {
    if (M <= 0 || N <= 0 || N % 4 != 0 || N > 512 || K % kBK != 0) return 1;
    const int64_t wgs = ((M + 63) / 64) * ((N + 63) / 64), steps = (K / kBK + 1) / 2;
    const int64_t s = std::min(std::min<int64_t>(256 / wgs, 16), std::min(steps / 4, max_part_bytes / (M * N * 4)));
    return s >= 2 && steps - steps / s >= 12 ? (int)s : 1;
}
int64_t skinny_part_rows(int64_t M, int N, int K) {
    const int64_t most = std::min(16, (K / kBK + 1) / 2 / 4);     // M * slices <= 64 * token tiles * (256 / workgroups)
    return M <= 0 || N <= 0 ? 0 : std::min(M * std::max<int64_t>(most, 1), std::max<int64_t>(M, 64 * 256 / ((N + 63) / 64)));
}

namespace {

// W where it lies: the k-split form
bool in_place(const GemmDesc& d) { return d.by_k || d.in_place; }

int launch_forms(const Call& c, hipStream_t st) {
    const GemmDesc& d = c.d;
    const bool by_k = c.b ? c.b->by_k : d.by_k;
    // 64 x 128 tiles once they alone fill the chip twice over; below that 64 x 64 tiles with a deep
    // ring (a narrower output has nothing to split: 32-token tiles, 128 columns)
    const int64_t wgs = ((d.M + 63) / 64) * ((d.N + 127) / 128);
    if (d.splits > 1) {                                                            // see skinny_splits
        if (d.dup2 == 2) return by_k ? launch_cfg<64, 64, 3, 2, true, 2, true>(c, st) : launch_cfg<64, 64, 3, 2, true, 2>(c, st);
        return by_k ? launch_cfg<64, 64, 3, 2, true, 1, true>(c, st) : launch_cfg<64, 64, 4, 2, true>(c, st);
    }
    if (d.dup2 == 2) {                                                             // see skinny_dup_applies
        // 128 columns per workgroup once that still puts a workgroup on every CU: the token tile is then fetched by
        // two workgroups instead of four (65B gate projection, inner rank 256: 2.16 -> 1.44 GB through the CUs,
        // backward 200 -> 157 us, forward 77 -> 62 us; three or four stages measure the same, two are slower)
        if (d.N > 64 && wgs >= 256) return by_k ? launch_cfg<64, 128, 3, 2, true, 2, true>(c, st) : launch_cfg<64, 128, 3, 2, true, 2>(c, st);
        return by_k ? launch_cfg<64, 64, 5, 2, true, 2, true>(c, st) : launch_cfg<64, 64, 5, 2, true, 2>(c, st);
    }
    if (in_place(d)) {                             // (whether B goes alone or beside A: the same tiles, so the same bits)
        if (d.N > 64 && wgs >= 256) return by_k ? launch_cfg<64, 128, 3, 2, true, 1, true>(c, st) : launch_cfg<64, 128, 3, 2, true>(c, st);
        return by_k ? launch_cfg<64, 64, 4, 2, true, 1, true>(c, st) : launch_cfg<64, 64, 4, 2, true>(c, st);
    }
    if (wgs >= 512) return launch_cfg<64, 128, 4, 1, false>(c, st);
    if (d.N > 64) return launch_cfg<64, 64, 5, 2, true>(c, st);
    return launch_cfg<32, 128, 6, 1, false>(c, st);
}

// what launch_forms decides by
bool same_form(const GemmDesc& a, const GemmDesc& b) {
    return a.M == b.M && a.N == b.N && a.dup2 == b.dup2 && (a.splits > 1) == (b.splits > 1) && !a.by_k && in_place(a) == in_place(b);
}

}  // namespace

int launch_skinny(const GemmDesc& d, hipStream_t st) { return launch_forms(Call{d, nullptr, nullptr, nullptr}, st); }

bool skinny_shares(const GemmDesc& d) { return d.by_k && skinny_applies(d); }
int launch_skinny_with(const GemmDesc& d, const PrepDesc& prep, const DequantDesc* weight, hipStream_t st) {
    if (!skinny_shares(d) || (weight && d.splits <= 1)) return QBLORA_ERR_UNSUPPORTED;
    return launch_forms(Call{d, nullptr, prep.blocks() ? &prep : nullptr, weight}, st);
}

int launch_skinny_pair(const GemmDesc& a, const GemmDesc& b, hipStream_t st) {
    if (skinny_applies(a) && skinny_applies(b) && same_form(a, b) && (a.splits <= 1 || a.part != b.part))
        return launch_forms(Call{a, &b, nullptr, nullptr}, st);
    const int rc = launch_gemm(a, st);
    return rc ? rc : launch_gemm(b, st);
}

}  // namespace qblora
