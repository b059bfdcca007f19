// Mid-batch forward of a 4-bit block-quantized layer without adapter (merged-model inference, Sec. 3.3, with
// a few dozen to 256 tokens in flight):
//
//   Y[t, n] = sum_k X[t, k] * w~[n, k],   w~ = bf16( c[code] * alpha (+ beta) )   (Eq. 1, the bf16 compute
//                                                                                  weight of the training forward)
//
// The regime: every weight is used T times, so up to a few dozen tokens the weight stream from HBM (0.5 byte
// of codes + the block parameters per weight) sets the time and at 128 tokens the MFMAs do.  A token tile of
// 256 (the training kernel) would waste most of its MFMAs here and, with one workgroup per 256 output rows,
// leave most of the chip idle.  Here a workgroup of 4 waves owns 128 output rows (32 per wave), ALL tokens
// (32 * TB of them, TB = 1 .. 5, to 8 in k_w4_wide) and one slice of the input dimension; the slices of a row tile (split-K, as
// many as the chip takes at once, see w4_mid_call_splits) write fp32 partial tiles that a second kernel adds in
// slice order (deterministic).
//
// A wave dequantizes its own MFMA operand in registers: lane l owns row (l & 31) and the 32 inputs
// 32*(l >> 5) .. +31 of each 64-input step, i.e. 16 bytes of codes, fetched with one load instruction (in the
// tile-ordered code copy the 32 rows of a step are adjacent: 1 KB contiguous per wave); dword j of them is the
// A operand (32 rows x 16 inputs, 8 per lane) of the j-th v_mfma_f32_32x32x16_bf16 of the step.  The weight
// tile never crosses LDS.  The token tile does ([token][64 inputs] bf16, 16-byte chunks XOR-swizzled by
// (row ^ row>>3) & 7): it is shared by the four waves, arrives by direct global -> LDS copies into a ring of
// four stages, and is read as the B operand (lane l: token l & 31, the same 8 inputs).  All vector-memory
// operations of the loop are issued from assembly statements three steps ahead (codes: four) and counted by
// hand (the compiler would tie every LDS access to them): a step waits until only the two youngest batches (the codes
// and the token tile of a step each) are outstanding.  The operands of step s+1 are built between the MFMAs of step s.
//
// From 161 tokens four waves copy and four contract (k_w4_wide).  Above 128 tokens one launch reads and dequantizes every weight once for all of them; two chunks of 128 did it twice (201
// tokens of 5120 x 13824 63 + 10 us for the contraction and the sum of the slices, one launch 47 + 5).  What bounds it: the
// partial tiles (256 workgroups of 128 rows x 256 tokens write and read 34 MB, about 14 us of 4096 x 4096's 23), then the
// matrix pipe at half to two thirds of its rate.
//
// A lane ends up with 4 consecutive output rows of one token per accumulator quad and stores them as one
// 8-byte word (bf16) or one 16-byte word (fp32 partials).
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace qblora {

namespace {

constexpr int kMidThreads = 256;
constexpr int kMidRows = 128;                   // output rows per workgroup
constexpr int kStages = 4;                      // ring of token tiles; operations are issued kStages - 1 steps ahead
constexpr int kTableReplicas = 8;

struct MidDesc {
    const uint8_t* codes; const float* scales; const float* beta; Codebook cb;
    int tiled;                 // codes (and, with 64-blocks, scales and offsets) in tile order
    int d_out, d_in;
    const qblora_bf16* X; int T;
    qblora_bf16* Y;            // splits == 1
    float* part;               // splits > 1: [splits][T][d_out] fp32
    int splits, steps_per_split;
};

__device__ __forceinline__ void copy16_to_lds(const void* uniform_base, uint32_t lane_offset, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_base), "v"(lane_offset), "s"(uniform_base) : "memory");
}
// The data of these loads arrive asynchronously: a destination may only be used behind a wait_slot that names it.
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
__device__ __forceinline__ void load16(u32x4& v, uint32_t lane_offset, const void* uniform_base) {
    asm volatile("global_load_dwordx4 %0, %1, %2" : "=&v"(v) : "v"(lane_offset), "s"(uniform_base) : "memory");
}
__device__ __forceinline__ void load4(float& v, uint32_t lane_offset, const void* uniform_base) {
    asm volatile("global_load_dword %0, %1, %2" : "=&v"(v) : "v"(lane_offset), "s"(uniform_base) : "memory");
}
__device__ __forceinline__ void load16f(f32x4& v, uint32_t lane_offset, const void* uniform_base) {
    asm volatile("global_load_dwordx4 %0, %1, %2" : "=&v"(v) : "v"(lane_offset), "s"(uniform_base) : "memory");
}

__device__ __forceinline__ uint32_t lds_address(const void* p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

// codes and block parameters of one step, as fetched
template <int BR>
struct Slot {
    u32x4 cw;
    float sc, be;              // 64-blocks: the row's scale and offset of this step
    f32x4 sc4, be4;            // 8 x 8 blocks: those of the lane's four block columns
    f32x4 sc4b, be4b;          // blocks of 8 rows x 4 inputs (BR = 84): the lane has eight block columns, these are 4 .. 7
};

template <int N, int BR, bool BETA>
__device__ __forceinline__ void wait_slot(Slot<BR>& s) {
    if constexpr (BR == 84) {
        if constexpr (BETA)
            asm volatile("s_waitcnt vmcnt(%5)" : "+v"(s.cw), "+v"(s.sc4), "+v"(s.sc4b), "+v"(s.be4), "+v"(s.be4b) : "n"(N) : "memory");
        else asm volatile("s_waitcnt vmcnt(%3)" : "+v"(s.cw), "+v"(s.sc4), "+v"(s.sc4b) : "n"(N) : "memory");
    } else if constexpr (BR == 8) {
        if constexpr (BETA) asm volatile("s_waitcnt vmcnt(%3)" : "+v"(s.cw), "+v"(s.sc4), "+v"(s.be4) : "n"(N) : "memory");
        else asm volatile("s_waitcnt vmcnt(%2)" : "+v"(s.cw), "+v"(s.sc4) : "n"(N) : "memory");
    } else {
        if constexpr (BETA) asm volatile("s_waitcnt vmcnt(%3)" : "+v"(s.cw), "+v"(s.sc), "+v"(s.be) : "n"(N) : "memory");
        else asm volatile("s_waitcnt vmcnt(%2)" : "+v"(s.cw), "+v"(s.sc) : "n"(N) : "memory");
    }
}

// How a code becomes a number: any codebook through a table of byte pairs in LDS, the codebook 0, 1, ..., 15 by byte
// conversions, and the same with the nibbles of every code dword regrouped by the decode pack (64-blocks).
enum { TABLE, INT4, REGROUPED };

// Rows nb .. nb + 3 of token `tok`: a slice's partial sums, or the output
__device__ __forceinline__ void store_four(const MidDesc& d, int z, int nb, int tok, const f32x4& v) {
    const int d_out = d.d_out;
    if (tok >= d.T || nb >= d_out) return;
    const bool whole = (d_out & 3) == 0;
    if (d.splits > 1) {
        float* p = d.part + ((int64_t)z * d.T + tok) * d_out + nb;
        if (whole) { *reinterpret_cast<f32x4*>(p) = v; return; }
        p[0] = v[0];
        if (nb + 1 < d_out) p[1] = v[1];
        if (nb + 2 < d_out) p[2] = v[2];
        if (nb + 3 < d_out) p[3] = v[3];
    } else {
        uint16_t* p = reinterpret_cast<uint16_t*>(d.Y) + (int64_t)tok * d_out + nb;
        const uint32_t lo = pack_bf16(v[0], v[1]), hi = pack_bf16(v[2], v[3]);
        if (whole) { *reinterpret_cast<uint2*>(p) = make_uint2(lo, hi); return; }
        p[0] = (uint16_t)(lo & 0xffffu);
        if (nb + 1 < d_out) p[1] = (uint16_t)(lo >> 16);
        if (nb + 2 < d_out) p[2] = (uint16_t)(hi & 0xffffu);
        if (nb + 3 < d_out) p[3] = (uint16_t)(hi >> 16);
    }
}

// TB: 32-token blocks; BETA: offsets present; BR: 1 (64 inputs of one row), 8 (8 rows x 8 inputs) or 84 (8 rows x 4 inputs)
template <int TB, bool BETA, int BR, int CODES>
__global__ __launch_bounds__(kMidThreads) void k_w4_mid(MidDesc d) {
    static_assert(CODES != REGROUPED || (BETA && BR == 1), "regrouped codes belong to INT4 models in 64-blocks");
    constexpr int kStageBytes = TB * 32 * 128;
    static_assert(BR == 1 || BR == 8 || BR == 84, "block shape");
    constexpr int kParamLoads = BR == 84 ? 2 : 1;              // 16-byte (or 4-byte) loads of scales per step; as many of offsets
    constexpr int kOps = TB + 1 + kParamLoads * (BETA ? 2 : 1);   // vector-memory operations per wave and step
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* const sX = smem;                                              // kStages token tiles
    float2* const sT = reinterpret_cast<float2*>(smem + kStages * kStageBytes);  // byte -> (c[lo], c[hi]), replicated

    const int d_out = d.d_out, d_in = d.d_in, T = d.T;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int r = lane & 31, h = lane >> 5;
    const int tiles_n = (d_out + kMidRows - 1) / kMidRows;
    const int nt = blockIdx.x % tiles_n, z = blockIdx.x / tiles_n;
    const int n0 = nt * kMidRows + wave * 32;
    const int n = min(n0 + r, d_out - 1);                       // rows past the end are computed, never stored
    const int steps_total = d_in / kBlock;
    const int s_begin = z * d.steps_per_split;
    const int s_end = min(steps_total, s_begin + d.steps_per_split);

    if constexpr (CODES == TABLE) {
        const float2 e = make_float2(d.cb.c[t & 15], d.cb.c[t >> 4]);
#pragma unroll
        for (int q = 0; q < kTableReplicas; ++q) sT[t * kTableReplicas + q] = e;
    }
    const float2* const my_table = sT + (lane & (kTableReplicas - 1));

    // ---- addresses: per-lane byte offsets are fixed, the wave-uniform bases walk along the steps --------------
    const int64_t bpr = steps_total;
    const int64_t run = d.tiled ? (((int64_t)(n >> 8) * bpr) * 256 + (n & 255)) : (int64_t)n * bpr;   // block 0 of row n
    const int64_t bstep = d.tiled ? 256 : 1;                                                          // next block
    const uint32_t c_off = (uint32_t)(run * 32 + 16 * h);
    uint32_t s_off;
    int64_t s_step;                                            // bytes per step in the scale / offset arrays
    if constexpr (BR == 84) {                                  // 16 block columns per step, the lane's half: 8
        s_off = (uint32_t)((((int64_t)(n >> 3) * (d_in >> 2)) + 8 * h) * 4);
        s_step = 64;
    } else if constexpr (BR == 8) {
        s_off = (uint32_t)((((int64_t)(n >> 3) * (d_in >> 3)) + 4 * h) * 4);
        s_step = 32;
    } else {
        s_off = (uint32_t)(run * 4);
        s_step = bstep * 4;
    }
    const int64_t c_step = bstep * 32;
    // copies of the token tile: wave w fills rows 8*TB*w .. +8*TB-1, copy i rows 8*(TB*w + i) + (lane >> 3)
    uint32_t x_off[TB];
#pragma unroll
    for (int i = 0; i < TB; ++i) {
        const int row = 8 * (TB * wave + i) + (lane >> 3);
        const int chunk = (lane & 7) ^ ((row ^ (row >> 3)) & 7);
        x_off[i] = (uint32_t)((int64_t)min(row, T - 1) * d_in * 2 + chunk * 16);
    }
    const uint32_t lds_x = __builtin_amdgcn_readfirstlane(lds_address(sX) + wave * TB * 1024);
    const unsigned char* const cbase = d.codes;
    const unsigned char* const sbase = reinterpret_cast<const unsigned char*>(d.scales);
    const unsigned char* const bbase = reinterpret_cast<const unsigned char*>(d.beta);
    const unsigned char* const xbase = reinterpret_cast<const unsigned char*>(d.X);

    // One batch of operations per step, the same count (kOps) whatever the step: the codes and block parameters of step
    // `sc` into register slot `sl` in front of the step's MFMAs, and the copies of the token tile of step `sx` into ring
    // stage `stage`, one behind every fourth of them.  Steps past the slice are redirected to its last step (fetched,
    // never used).
    auto issue_codes = [&](Slot<BR>& sl, int step) __attribute__((always_inline)) {
        const int64_t sc = min(step, s_end - 1);
        load16(sl.cw, c_off, cbase + sc * c_step);
        if constexpr (BR == 84) {
            load16f(sl.sc4, s_off, sbase + sc * s_step);
            load16f(sl.sc4b, s_off + 16, sbase + sc * s_step);
            if constexpr (BETA) { load16f(sl.be4, s_off, bbase + sc * s_step); load16f(sl.be4b, s_off + 16, bbase + sc * s_step); }
        } else if constexpr (BR == 8) {
            load16f(sl.sc4, s_off, sbase + sc * s_step);
            if constexpr (BETA) load16f(sl.be4, s_off, bbase + sc * s_step);
        } else {
            load4(sl.sc, s_off, sbase + sc * s_step);
            if constexpr (BETA) load4(sl.be, s_off, bbase + sc * s_step);
        }
    };
    auto issue_x = [&](int step, int stage, int i) __attribute__((always_inline)) {
        const int64_t sx = min(step, s_end - 1);
        copy16_to_lds(xbase + sx * 128, x_off[i], lds_x + stage * kStageBytes + i * 1024);
    };

    // fragment addresses of the token tile: token 32*tb + r, logical chunk 4h + j
    uint32_t f_off[TB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
        const int row = 32 * tb + r;
        f_off[tb] = row * 128 + (((4 * h) ^ ((row ^ (row >> 3)) & 7)) << 4);
    }

    f32x16 acc[TB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[tb][i] = 0.0f;

    auto weight = [&](float c, float a, float b) __attribute__((always_inline)) {
        return BETA ? __fmaf_rn(c, a, b) : __fmul_rn(c, a);
    };
    // Dequantization in 16 units per step: unit k = 4j + i makes dword i (two weights, inputs 2i and 2i+1 of the
    // 8) of the j-th A operand (code dword j).  Table form: unit_a fetches the byte's (c[lo], c[hi]) pair from LDS,
    // unit_b scales, offsets and rounds.  The bytes of an INT4 model's (w & 0x0F0F0F0F) are inputs 0, 2, 4, 6 and those of
    // ((w >> 4) & 0x0F0F0F0F) 1, 3, 5, 7; a regrouped dword holds input 0, 2, 4, 6, 1, 3, 5, 7 in its nibbles, so there
    // they are inputs 0, 4, 1, 5 and 2, 6, 3, 7.
    struct Params { uint32_t cw[4]; float a[8], b[8]; };       // scale / offset of inputs 0..3 and 4..7 of each code dword
    auto params = [&](const Slot<BR>& sl) __attribute__((always_inline)) {
        Params p;
        p.cw[0] = sl.cw.x; p.cw[1] = sl.cw.y; p.cw[2] = sl.cw.z; p.cw[3] = sl.cw.w;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int j = e >> 1;
            if constexpr (BR == 84) {
                p.a[e] = e < 4 ? sl.sc4[e] : sl.sc4b[e - 4];
                p.b[e] = !BETA ? 0.0f : e < 4 ? sl.be4[e] : sl.be4b[e - 4];
            } else {
                p.a[e] = BR == 8 ? sl.sc4[j] : sl.sc;
                p.b[e] = !BETA ? 0.0f : BR == 8 ? sl.be4[j] : sl.be;
            }
        }
        return p;
    };
    auto unit_a = [&](const Params& p, int k, float2& tv) __attribute__((always_inline)) {
        if constexpr (CODES == TABLE) tv = my_table[((p.cw[k >> 2] >> (8 * (k & 3))) & 0xffu) * kTableReplicas];
    };
    auto unit_b = [&](const Params& p, int k, const float2& tv) __attribute__((always_inline)) {
        const int j = k >> 2, i = k & 3;
        float lo, hi;
        if constexpr (CODES == REGROUPED) {
            const uint32_t t = (p.cw[j] >> (4 * (i & 1))) & 0x0F0F0F0Fu;       // i odd: inputs 2, 6, 3, 7
            lo = (float)((t >> (8 * (i >> 1))) & 0xffu);                          // i < 2: bytes 0 and 2, else 1 and 3
            hi = (float)((t >> (16 + 8 * (i >> 1))) & 0xffu);
        } else if constexpr (CODES == INT4) {
            lo = (float)((p.cw[j] >> (8 * i)) & 15u);
            hi = (float)((p.cw[j] >> (8 * i + 4)) & 15u);
        } else {
            lo = tv.x; hi = tv.y;
        }
        const int e = 2 * j + (i >> 1);                        // byte i of the dword: inputs 2i, 2i+1
        return pack_bf16(weight(lo, p.a[e], p.b[e]), weight(hi, p.a[e], p.b[e]));
    };
    // all four operands at once (before the loop)
    auto dequantize = [&](const Slot<BR>& sl, bf16x8 (&wf)[4]) __attribute__((always_inline)) {
        const Params p = params(sl);
        uint32_t o[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) { float2 tv = make_float2(0.f, 0.f); unit_a(p, k, tv); o[k] = unit_b(p, k, tv); }
#pragma unroll
        for (int j = 0; j < 4; ++j) wf[j] = __builtin_bit_cast(bf16x8, make_uint4(o[4 * j], o[4 * j + 1], o[4 * j + 2], o[4 * j + 3]));
    };
    // One step: the 4 * TB MFMAs on this step's operands `wf`, and between them the units that build the next
    // step's operands `wn` from slot `sl` -- written in issue order and fenced after every MFMA: a wave issues in
    // order, so vector work has to sit between the MFMAs to run in their shadow.  LDS reads are issued two MFMAs (token
    // fragment; four or eight ahead measured the same) or one unit (table pair) ahead of their use.  The copies of a later
    // tile are spread over the step: a copy holds the address path for 16 cycles or more, and the waves' bursts of TB of
    // them in front of the MFMAs left the matrix pipe idle (22016 x 8192 at 256 tokens 120 -> 107 us, 11008 x 4096 42.6 ->
    // 38.6).
    auto step = [&](const bf16x8 (&wf)[4], int now, int stage, const Slot<BR>& sl, bf16x8 (&wn)[4]) __attribute__((always_inline)) {
        constexpr int M = 4 * TB;
        const unsigned char* xs = sX + stage * kStageBytes;
        const Params p = params(sl);
        uint32_t o[16];
        float2 tv[2] = {make_float2(0.f, 0.f), make_float2(0.f, 0.f)};
        bf16x8 xf[2];
        auto read_x = [&](int m) __attribute__((always_inline)) {
            return *reinterpret_cast<const bf16x8*>(xs + (f_off[m % TB] ^ ((m / TB) << 4)));
        };
        unit_a(p, 0, tv[0]);
#pragma unroll
        for (int m = 0; m < 2; ++m) xf[m] = read_x(m);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < M; ++m) {
            acc[m % TB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[m / TB], xf[m & 1], acc[m % TB], 0, 0, 0);
            if (m + 2 < M) xf[m & 1] = read_x(m + 2);
            if (m % 4 == 1) issue_x(now + kStages - 1, (stage + kStages - 1) % kStages, m / 4);
#pragma unroll
            for (int k = m * 16 / M; k < (m + 1) * 16 / M; ++k) {
                if (k + 1 < 16) unit_a(p, k + 1, tv[(k + 1) & 1]);
                o[k] = unit_b(p, k, tv[k & 1]);
                asm volatile("" : "+v"(o[k]));                  // computed here
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            wn[j] = __builtin_bit_cast(bf16x8, make_uint4(o[4 * j], o[4 * j + 1], o[4 * j + 2], o[4 * j + 3]));
    };

    Slot<BR> slot[kStages];
#pragma unroll
    for (int u = 0; u < kStages; ++u) {                         // defined values for the fields a variant never loads
        slot[u].sc = 0.0f; slot[u].be = 0.0f;
        slot[u].sc4 = f32x4{0.f, 0.f, 0.f, 0.f}; slot[u].be4 = f32x4{0.f, 0.f, 0.f, 0.f};
        slot[u].sc4b = f32x4{0.f, 0.f, 0.f, 0.f}; slot[u].be4b = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    bf16x8 wf[2][4];                                            // operands of this step and of the next
    __syncthreads();                                            // the table is complete
    // The weights of step s+1 are dequantized while the MFMAs of step s issue, so the codes run one step ahead of
    // the token tiles: batch b carries the codes of step b+4 and the tile of step b+3.
    issue_codes(slot[0], s_begin);
#pragma unroll
    for (int u = 0; u < kStages - 1; ++u) {
        issue_codes(slot[u + 1], s_begin + u + 1);
#pragma unroll
        for (int i = 0; i < TB; ++i) issue_x(s_begin + u, u, i);
    }
    wait_slot<(kStages - 1) * kOps, BR, BETA>(slot[0]);
    dequantize(slot[0], wf[0]);
    for (int s = s_begin; s < s_end; s += kStages) {
#pragma unroll
        for (int u = 0; u < kStages; ++u) {
            // the batch issued three steps ago is in when at most the two after it are outstanding
            wait_slot<(kStages - 2) * kOps, BR, BETA>(slot[(u + 1) % kStages]);
            __syncthreads();                                    // every wave's part of the tile is in; all waves are past
                                                                // the step before, whose stage this step refills
            issue_codes(slot[u], s + u + kStages);              // slot u was turned into operands a step ago
            if (s + u < s_end) step(wf[u & 1], s + u, u, slot[(u + 1) % kStages], wf[(u + 1) & 1]);
        }
    }
#pragma unroll
    for (int u = 0; u < kStages; ++u) wait_slot<0, BR, BETA>(slot[u]);     // the redirected look-ahead operations

    // ---- store: lane = token 32*tb + r; registers 4q .. 4q+3 = rows 8q + 4h .. +3 of the wave's 32 ----------
#pragma unroll
    for (int tb = 0; tb < TB; ++tb)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            store_four(d, z, n0 + 8 * q + 4 * h, 32 * tb + r, f32x4{acc[tb][4 * q], acc[tb][4 * q + 1], acc[tb][4 * q + 2], acc[tb][4 * q + 3]});
}

// The same layer on 161 to 256 tokens (TB = 6 .. 8).  A copy instruction holds up the wave that issues it, and one wave per SIMD
// contracts by v_mfma_f32_32x32x16_bf16 at little more than half of the pipe's rate, by 16x16x32 at nearly all of it.  Here four
// waves do nothing but copy, three the token tiles into a ring of four stages and one the codes, scales and offsets into a
// ring of its own, deeper because they come from HBM (waits are in order: beside tokens in one wave's queue they could not be).
// The other four read all of it from LDS and contract in 16 x 16 blocks; codes of INT4 models become floats two at a time.  One
// barrier a step.  Kernel us in the form above / here: 201 tokens of 5120 x 13824 INT4 40.4 / 37.3, 256 of 22016 x 8192 123 / 111,
// 256 of 4096 x 4096 20.2 / 18.3; codebooks 200 of 8192 x 8192 39.4 / 36.0, row-major 256 of 5120 x 13824 50.6 / 45.4; 161 of 11008 x
// 4096 in 8 x 8 blocks 30.9 / 30.0; 129 tokens of 22016 x 8192 79 / 81, so that five token blocks stay above.  What bounds it: LDS
// (128 KB of fragments and 37 KB of copies a step of 256 tokens) and the expansion, 300 cycles beside 1024 of MFMAs, that only
// partly hides: without it 256 of 22016 x 8192 take 106, without MFMAs 55.  (Eight waves that share the rows and halve the tokens
// expand twice: 134.)
template <int TB, int CODES, int BR>
struct Wide {
    static constexpr int kTokens = TB * 32 * 128;
    static constexpr int kParams = BR == 84 ? 1024 : 512;      // scales of 128 rows and a step, and again offsets
    static constexpr int kCodes = 4096 + 2 * kParams;
    static constexpr int kReplicas = TB == 8 ? 4 : kTableReplicas;
    static constexpr int kTable = CODES == TABLE ? 256 * kReplicas * (int)sizeof(float2) : 0;
    static constexpr int kRoom = (160 * 1024 - kStages * kTokens - kTable) / kCodes;
    static constexpr int kCodeStages = kRoom < 8 ? kRoom : 8;
    static constexpr int kXOps = (4 * TB + 2) / 3;             // copies of a token wave and step
    static constexpr int kLds = kStages * kTokens + kCodeStages * kCodes + kTable;
    static_assert(kCodeStages >= 4, "codes in flight");
};

__device__ __forceinline__ void gather16_to_lds(const unsigned char* p, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(lds_base), "v"(p) : "memory");
}
__device__ __forceinline__ void gather4_to_lds(const unsigned char* p, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" :: "s"(lds_base), "v"(p) : "memory");
}

constexpr int kWideThreads = 512;

template <int TB, bool BETA, int BR, int CODES>
__global__ __launch_bounds__(kWideThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_w4_wide(MidDesc d) {
    static_assert(CODES != REGROUPED || (BETA && BR == 1), "regrouped codes belong to INT4 models in 64-blocks");
    typedef Wide<TB, CODES, BR> G;
    constexpr int CS = G::kCodeStages;
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* const sC = smem + kStages * G::kTokens;                       // codes and block parameters
    float2* const sT = reinterpret_cast<float2*>(sC + CS * G::kCodes);           // byte -> (c[lo], c[hi]), replicated

    const int d_out = d.d_out, d_in = d.d_in, T = d.T;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int tiles_n = (d_out + kMidRows - 1) / kMidRows;
    const int nt = blockIdx.x % tiles_n, z = blockIdx.x / tiles_n;
    const int steps_total = d_in / kBlock;
    const int s_begin = z * d.steps_per_split;
    const int n = min(steps_total, s_begin + d.steps_per_split) - s_begin;       // steps of this slice, at least one

    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem));
    // Copying waves: steps past the slice are redirected to its last one (fetched, never used), so that the counts stay.
    if (wave >= 5) {
        // ---- tokens: wave c fetches eight rows with each of its copies c, c + 3, ... (some the last ones again) --------------
        constexpr int kXOps = G::kXOps;
        const int c = wave - 5;
        uint32_t x_off[kXOps];
#pragma unroll
        for (int i = 0; i < kXOps; ++i) {
            const int row = 8 * min(c + 3 * i, 4 * TB - 1) + (lane >> 3);
            // chunk c of a row sits at (4*(c & 1) + (c >> 1)) ^ (row >> 1 & 7): the sixteen rows of a fragment touch every bank
            // once, and a lane's two chunks of a step are neighbours in the row, like its codes
            const int v = (lane & 7) ^ ((row >> 1) & 7), chunk = 2 * (v & 3) + (v >> 2);
            x_off[i] = (uint32_t)((int64_t)min(row, T - 1) * d_in * 2 + chunk * 16);
        }
        const unsigned char* const xbase = reinterpret_cast<const unsigned char*>(d.X) + (int64_t)s_begin * 128;
        auto issue = [&](int s) __attribute__((always_inline)) {
            const int64_t at = min(s, n - 1);
#pragma unroll
            for (int i = 0; i < kXOps; ++i)
                copy16_to_lds(xbase + at * 128, x_off[i], lds0 + (s % kStages) * G::kTokens + min(c + 3 * i, 4 * TB - 1) * 1024);
        };
#pragma unroll
        for (int u = 0; u < kStages - 1; ++u) issue(u);
        asm volatile("s_barrier" ::: "memory");                // (the codes)
#pragma unroll 1
        for (int s = 0; s < n; ++s) {
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"((kStages - 2) * kXOps) : "memory");   // step s is in, all are past s - 1
            issue(s + kStages - 1);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // nothing may arrive behind the workgroup's end
        return;
    }
    if (wave == 4) {
        // ---- codes and block parameters of the 128 rows; rows past the end are computed, never stored ----------------------
        const int row0 = nt * kMidRows;
        const int64_t bpr = steps_total, bstep = d.tiled ? 256 : 1;
        auto block_of = [&](int row) { return d.tiled ? ((int64_t)(row >> 8) * bpr) * 256 + (row & 255) : (int64_t)row * bpr; };
        const unsigned char* codes[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            codes[i] = d.codes + (block_of(min(row0 + 32 * i + (lane >> 1), d_out - 1)) + s_begin * bstep) * 32 + 16 * (lane & 1);
        // 16 bytes a lane, scales then offsets; row-major 64-blocks: 4 bytes
        constexpr int kP = BR == 84 ? 2 : BR == 1 ? 4 : 1;
        constexpr int per = BR == 84 ? 4 : 2, cols = BR == 84 ? 4 : 8;         // 16-byte pieces of a block row and step; inputs a block
        const unsigned char* params[kP];
#pragma unroll
        for (int i = 0; i < kP; ++i) {
            int64_t at;
            bool scales;
            if constexpr (BR == 1) {
                scales = d.tiled ? lane < 32 : i < 2;
                at = (d.tiled ? block_of(min(row0 + 4 * (lane & 31), (d_out - 1) & ~3)) : block_of(min(row0 + 64 * (i & 1) + lane, d_out - 1))) + s_begin * bstep;
            } else {
                const int u = (64 * i + lane) % (16 * per);
                scales = 64 * i + lane < 16 * per;
                at = (int64_t)min((row0 >> 3) + u / per, (d_out >> 3) - 1) * (d_in / cols) + 4 * (u % per) + (int64_t)s_begin * (64 / cols);
            }
            params[i] = reinterpret_cast<const unsigned char*>((scales || !BETA ? d.scales : d.beta) + at);
        }
        const int64_t p_step = BR == 1 ? bstep * 4 : 64 / cols * 4;
        const uint32_t lds_c = lds0 + kStages * G::kTokens;
        auto run = [&](auto four) __attribute__((always_inline)) {             // four: 4-byte fetches
            constexpr bool kFour = BR == 1 && four.value;
            constexpr int kParamOps = kFour ? 4 : BR == 84 ? 2 : 1, kOps = 4 + kParamOps;
            static_assert((CS - 1) * kOps < 64, "six bits of the wait counter");
            auto issue = [&](int s, int slot) __attribute__((always_inline)) {
                const int64_t at = min(s, n - 1);
                const uint32_t to = lds_c + slot * G::kCodes;
#pragma unroll
                for (int i = 0; i < 4; ++i) gather16_to_lds(codes[i] + at * bstep * 32, to + i * 1024);
#pragma unroll
                for (int i = 0; i < kParamOps; ++i) {
                    if constexpr (kFour) gather4_to_lds(params[i] + at * p_step, to + 4096 + i * 256);
                    else gather16_to_lds(params[i] + at * p_step, to + 4096 + i * 1024);
                }
            };
#pragma unroll 1
            for (int u = 0; u < CS; ++u) issue(u, u);
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"((CS - 1) * kOps) : "memory");      // the first are in
            int slot = 0;
#pragma unroll 1
            for (int s = 0; s < n; ++s) {
                asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"((CS - 2) * kOps) : "memory");  // those of step s + 1 are
                issue(s + CS, slot);                           // the codes of step s were expanded a step ago
                slot = slot + 1 == CS ? 0 : slot + 1;
            }
        };
        if (BR == 1 && !d.tiled) run(std::true_type{}); else run(std::false_type{});
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        return;
    }

    if constexpr (CODES == TABLE) {
        const float2 e = make_float2(d.cb.c[t & 15], d.cb.c[t >> 4]);
#pragma unroll
        for (int q = 0; q < G::kReplicas; ++q) sT[t * G::kReplicas + q] = e;
    }
    const float2* const my_table = sT + (lane & (G::kReplicas - 1));
    // fragment of 16 tokens and a slice ks of 32 inputs: lane (r, g) reads chunk 2g + ks of token r
    const uint32_t x_at = (uint32_t)(r * 128 + ((g ^ (r >> 1)) << 4));
    constexpr int NT = 2 * TB;                                 // 16-token blocks
    f32x4 acc[2][NT];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int tb = 0; tb < NT; ++tb) acc[b][tb] = f32x4{0.f, 0.f, 0.f, 0.f};

    // codes of the lane's 16 inputs (16g .. +15 of the step) of rows r and 16 + r, and their scales and offsets
    struct Params { uint2 cw[2]; f32x4 a[2], b[2]; };
    auto load_params = [&](int slot) __attribute__((always_inline)) {
        const unsigned char* const p = sC + slot * G::kCodes + wave * 1024;
        const unsigned char* const q = sC + slot * G::kCodes + 4096 + wave * (G::kParams / 4);
        Params v;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int row = 16 * b + r;
            v.cw[b] = *reinterpret_cast<const uint2*>(p + row * 32 + 8 * g);
            auto values = [&](const unsigned char* at) __attribute__((always_inline)) {
                f32x4 f = {0.f, 0.f, 0.f, 0.f};
                if constexpr (BR == 1) {
                    f[0] = *reinterpret_cast<const float*>(at + row * 4);
                } else if constexpr (BR == 8) {
                    const float2 two = *reinterpret_cast<const float2*>(at + (row >> 3) * 32 + 8 * g);
                    f[0] = two.x; f[1] = two.y;
                } else {
                    f = *reinterpret_cast<const f32x4*>(at + (row >> 3) * 64 + 16 * g);
                }
                return f;
            };
            v.a[b] = values(q);
            if constexpr (BETA) v.b[b] = values(q + G::kParams); else v.b[b] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        return v;
    };
    // unit k = 8b + 4ks + i: dword i (inputs 2i, 2i + 1 of eight) of the operand of rows 16b .. and slice ks
    auto word_of = [&](const Params& p, int k) __attribute__((always_inline)) { return (k >> 2) & 1 ? p.cw[k >> 3].y : p.cw[k >> 3].x; };
    auto unit_a = [&](const Params& p, int k, float2& tv) __attribute__((always_inline)) {
        if constexpr (CODES == TABLE) tv = my_table[((word_of(p, k) >> (8 * (k & 3))) & 0xffu) * G::kReplicas];
    };
    f32x2 f_lo[2], f_hi[2];                                    // converted codes of units under way
    auto unit_b = [&](const Params& p, int k, const float2& tv) __attribute__((always_inline)) {
        const int b = k >> 3, ks = (k >> 2) & 1, i = k & 3;
        const uint32_t w = word_of(p, k);
        float lo, hi;
        if constexpr (CODES == TABLE) {
            lo = tv.x; hi = tv.y;
        } else {
            // a nibble as an E4M3 number is the code times 2^-9: two codes a conversion, exact.  Of the eight nibbles, low
            // ones first in each byte: inputs 0, 1, 2, ..., or regrouped 0, 2, 4, 6, 1, 3, 5, 7.
            constexpr bool kPairs = CODES == REGROUPED;        // a byte pair gives the low or high inputs of two units
            if (kPairs ? i < 2 : i % 2 == 0) {
                if constexpr (kPairs) {
                    const uint32_t v = (w >> (4 * i)) & 0x0F0F0F0Fu;
                    f_lo[i] = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(v, 512.0f, false);
                    f_hi[i] = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(v, 512.0f, true);
                } else {
                    const uint32_t e = w & 0x0F0F0F0Fu, q = (w >> 4) & 0x0F0F0F0Fu;
                    f_lo[0] = i ? __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(e, 512.0f, true) : __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(e, 512.0f, false);
                    f_hi[0] = i ? __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(q, 512.0f, true) : __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(q, 512.0f, false);
                }
            }
            const int at = kPairs ? i & 1 : 0, el = kPairs ? i >> 1 : i & 1;
            lo = f_lo[at][el]; hi = f_hi[at][el];
        }
        const int e = BR == 84 ? 2 * ks + (i >> 1) : BR == 8 ? ks : 0;
        const float sc = p.a[b][e], of = p.b[b][e];
        return BETA ? pack_bf16(__fmaf_rn(lo, sc, of), __fmaf_rn(hi, sc, of)) : pack_bf16(__fmul_rn(lo, sc), __fmul_rn(hi, sc));
    };
    auto operands = [&](const uint32_t (&o)[16], bf16x8 (&wf)[4]) __attribute__((always_inline)) {      // wf[2b + ks]
#pragma unroll
        for (int j = 0; j < 4; ++j) wf[j] = __builtin_bit_cast(bf16x8, make_uint4(o[4 * j], o[4 * j + 1], o[4 * j + 2], o[4 * j + 3]));
    };
    // One step: the MFMAs on operands `wf`, and between them the next step's operands `wn` from code stage `slot`; written in
    // issue order and fenced, LDS reads ahead of their use, as in k_w4_mid.  A fragment serves both row blocks.
    auto step = [&](const bf16x8 (&wf)[4], int stage, int slot, bf16x8 (&wn)[4]) __attribute__((always_inline)) {
        constexpr int M = 4 * NT, kAhead = 3;
        const unsigned char* xs = smem + stage * G::kTokens;
        auto read_x = [&](int f) __attribute__((always_inline)) {             // fragment f = ks * NT + tb
            return *reinterpret_cast<const bf16x8*>(xs + (x_at ^ (uint32_t)((f / NT) << 6)) + (f % NT) * 2048);
        };
        const Params p = load_params(slot);
        bf16x8 xf[kAhead + 1];
#pragma unroll
        for (int f = 0; f < kAhead; ++f) xf[f] = read_x(f);
        uint32_t o[16];
        float2 tv[2] = {make_float2(0.f, 0.f), make_float2(0.f, 0.f)};
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const int f = m / 2, b = m & 1, ks = f / NT, tb = f % NT;
            acc[b][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[2 * b + ks], xf[f % (kAhead + 1)], acc[b][tb], 0, 0, 0);
            if (b == 0 && f + kAhead < M / 2) xf[(f + kAhead) % (kAhead + 1)] = read_x(f + kAhead);
            // the first MFMAs cover the reads of the codes: the sixteen units sit behind the others
            constexpr int kSkip = 6;
            const int k0 = m < kSkip ? 0 : (m - kSkip) * 16 / (M - kSkip), k1 = m < kSkip ? 0 : (m - kSkip + 1) * 16 / (M - kSkip);
            if (m == kSkip - 1) unit_a(p, 0, tv[0]);
#pragma unroll
            for (int k = k0; k < k1; ++k) {
                if (k + 1 < 16) unit_a(p, k + 1, tv[(k + 1) & 1]);
                o[k] = unit_b(p, k, tv[k & 1]);
                asm volatile("" : "+v"(o[k]));                  // computed here
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        operands(o, wn);
    };
    auto top = [&]() __attribute__((always_inline)) {          // this wave's reads are done; what the step needs is in
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    bf16x8 wf[2][4];
    top();                                                     // the table is complete, the first codes are in
    {
        const Params p = load_params(0);
        uint32_t o[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) { float2 tv = make_float2(0.f, 0.f); unit_a(p, k, tv); o[k] = unit_b(p, k, tv); }
        operands(o, wf[0]);
    }
    int stage = 0, slot = 1;                                   // of the step's tokens and the next step's codes
    auto advance = [&]() __attribute__((always_inline)) {
        stage = (stage + 1) % kStages;
        slot = slot + 1 == CS ? 0 : slot + 1;
    };
    int s = 0;
    for (; s + 1 < n; s += 2) {
        top();
        step(wf[0], stage, slot, wf[1]);
        advance();
        top();
        step(wf[1], stage, slot, wf[0]);
        advance();
    }
    if (s < n) {
        top();
        step(wf[0], stage, slot, wf[1]);
    }

    // ---- store: the lane holds token 16*tb + r, rows 16*b + 4*g .. +3 of the wave's 32 ---------------------------------
    const int n0 = nt * kMidRows + wave * 32;
#pragma unroll
    for (int tb = 0; tb < NT; ++tb)
#pragma unroll
        for (int b = 0; b < 2; ++b) store_four(d, z, n0 + 16 * b + 4 * g, 16 * tb + r, acc[b][tb]);
}

// Y = bf16( sum_z part[z] ), slices added in ascending order, four outputs per thread (Y is 8-byte aligned)
__global__ __launch_bounds__(256) void k_w4_mid_reduce(const float* __restrict__ part, int splits, int64_t count,
                                                       qblora_bf16* __restrict__ Y) {
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (i >= count) return;
    if ((count & 3) == 0) {                                     // every slice's words are aligned
        f32x4 s = *reinterpret_cast<const f32x4*>(part + i);
        for (int z0 = 1; z0 < splits; z0 += 4) {                // four slices' loads issued together
            f32x4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const f32x4*>(part + min(z0 + u, splits - 1) * count + i);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (z0 + u < splits) s += v[u];
        }
        *reinterpret_cast<uint2*>(Y + i) = make_uint2(pack_bf16(s[0], s[1]), pack_bf16(s[2], s[3]));
        return;
    }
    for (int e = 0; e < 4 && i + e < count; ++e) {
        float a = 0.0f;
        for (int zz = 0; zz < splits; ++zz) a += part[zz * count + i + e];
        reinterpret_cast<uint16_t*>(Y)[i + e] = (uint16_t)(pack_bf16(a, a) & 0xffffu);
    }
}

template <int TB>
constexpr size_t mid_lds(int codes) {
    return (size_t)kStages * TB * 32 * 128 + (codes == TABLE ? 256 * kTableReplicas * sizeof(float2) : 0);
}

template <typename K>
bool set_lds(K kernel, size_t smem) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)smem) == hipSuccess;
}

template <int TB, bool BETA, int BR, int CODES>
int launch_one(const MidDesc& d, unsigned blocks, hipStream_t st) {
    if constexpr (TB > 5) {
        constexpr size_t smem = Wide<TB, CODES, BR>::kLds;
        static const bool ok = set_lds(k_w4_wide<TB, BETA, BR, CODES>, smem);
        if (!ok) return QBLORA_ERR_LAUNCH;
        hipLaunchKernelGGL((k_w4_wide<TB, BETA, BR, CODES>), dim3(blocks), dim3(kWideThreads), smem, st, d);
    } else {
        constexpr size_t smem = mid_lds<TB>(CODES);
        static const bool ok = set_lds(k_w4_mid<TB, BETA, BR, CODES>, smem);
        if (!ok) return QBLORA_ERR_LAUNCH;
        hipLaunchKernelGGL((k_w4_mid<TB, BETA, BR, CODES>), dim3(blocks), dim3(kMidThreads), smem, st, d);
    }
    return launch_status();
}

template <int TB, int BR>
int launch_br(const MidDesc& d, unsigned blocks, hipStream_t st, int form) {
    if constexpr (BR == 1)
        if (form == REGROUPED) return launch_one<TB, true, BR, REGROUPED>(d, blocks, st);
    if (form == INT4) return launch_one<TB, true, BR, INT4>(d, blocks, st);
    return d.beta ? launch_one<TB, true, BR, TABLE>(d, blocks, st) : launch_one<TB, false, BR, TABLE>(d, blocks, st);
}

template <int TB>
int launch_tb(const MidDesc& d, unsigned blocks, hipStream_t st, int form, int block_rows, int block_cols) {
    if (block_rows == 8 && block_cols == 4) return launch_br<TB, 84>(d, blocks, st, form);
    if (block_rows == 8) return launch_br<TB, 8>(d, blocks, st, form);
    return launch_br<TB, 1>(d, blocks, st, form);
}

}  // namespace

namespace {

// 32-token blocks of a workgroup: as many as there are (with two, four, six or eight of them alone 201 tokens of 5120 x
// 13824 took 48.0 us instead of 45.1, 129 of 22016 x 8192 88.7 instead of 74.5; with two codebook weights of 19200 x 13824
// take 49.2 at 17 tokens, with one 47.5)
int token_blocks(int T) { return (T + 31) / 32; }

// no empty slice, at least 4 steps each
int slices_of(int want, int steps) {
    want = std::max(std::min({want, steps / 4, 8}), 1);
    const int per = (steps + want - 1) / want;
    return (steps + per - 1) / per;
}

}  // namespace

// The most slices of the input dimension.  Up to 128 tokens, measured over 2 / 3 / 4 waves per workgroup and 1 .. 8 slices
// on 4096 x 4096, 11008 x 4096 and 22016 x 8192: what counts is the number of workgroups -- about 700 up to 64 tokens
// (the weight stream wants loads in flight), about 400 at 128 (two resident per CU; more slices only add partial
// tiles) -- while 64- or 96-row workgroups differ from 128-row ones by a few percent at most; one slice per row tile,
// which the balance of matrix work alone would choose at 128 tokens, is 20 % slower than two.  Above 128 tokens a
// workgroup's ring of token tiles takes a CU's LDS: as many slices as one round of 256 workgroups holds (measured with
// k_w4_mid, not again with k_w4_wide).
int w4_mid_splits(int d_out, int d_in, int T) {
    const int tiles_n = (d_out + kMidRows - 1) / kMidRows, target = T > 64 ? 400 : 700;
    return slices_of(T > 128 ? 256 / tiles_n : (target + tiles_n / 2) / tiles_n, d_in / kBlock);
}

// The slices of a call.  A codebook in LDS wants two workgroups on a CU up to 128 tokens, which w4_mid_splits counts on.
// Without one a lone workgroup hides its expansion nearly as well, so a step on two to a CU takes 1.6 times as long as on one,
// and a slice costs its partial tiles, a step per 2000 outputs.  us of 1 / 2 / 3 / 4 / 5 / 6 slices, packed INT4: 8192 x 8192 at 65
// tokens 54.9 / 34.1 / 26.9 / 23.3 / 27.2 / 26.3 (4: 256 workgroups), 5120 x 13824 88.7 / 50.3 / 36.3 / 29.8 / 26.2 / 24.1,
// 11008 x 13824 91.2 / 54.3 / 57.6 / 48.1 / 43.7 / 50.5, 22016 x 13824 at 97 103.0 / 98.7 / 109.3 / 97.2 / 100.0 / 108.4.  The least
// of this over the slices that the workspace counts on: over 1375 calls 0.7 % behind the best choice.
int w4_mid_call_splits(int d_out, int d_in, int T, bool table) {
    const int most = w4_mid_splits(d_out, d_in, T);
    if (table || T <= 64 || T > 128) return most;
    const int tiles_n = (d_out + kMidRows - 1) / kMidRows, steps = d_in / kBlock;
    int splits = most, best = 0;
    for (int want = 1; want <= most; ++want) {
        const int s = slices_of(want, steps), per = (steps + s - 1) / s, blocks = tiles_n * s;
        const int cost = per * (blocks <= 256 ? 10 : 16 * ((blocks + 511) / 512)) + (s > 1 ? s * d_out / 200 : 0);
        if (best == 0 || cost < best) { splits = s; best = cost; }
    }
    return splits;
}

size_t w4_mid_part_bytes(int d_out, int d_in, int T) {
    const int splits = w4_mid_splits(d_out, d_in, T);
    return splits > 1 ? sizeof(float) * (size_t)splits * (size_t)T * (size_t)d_out : 0;
}

int launch_w4_mid(const uint8_t* codes, const float* scales, const float* beta, const Codebook& cb, int tiled, int d_out,
                  int d_in, const qblora_bf16* X, int T, qblora_bf16* Y, float* part, hipStream_t st, int block_rows,
                  int regrouped, int block_cols) {
    if (T < 1 || T > 256 || d_in % kBlock != 0 || d_out < 1) return QBLORA_ERR_SHAPE;
    // 32-bit lane offsets: the arrays of one weight and the token rows must stay below 4 GiB
    if ((int64_t)((d_out + 255) / 256) * 256 * (d_in / 2) >= ((int64_t)1 << 32) || (int64_t)T * d_in * 2 >= ((int64_t)1 << 32))
        return QBLORA_ERR_SHAPE;
    if (block_rows == 8 && (d_out % 8 != 0)) return QBLORA_ERR_SHAPE;
    if (regrouped && (!beta || block_rows == 8)) return QBLORA_ERR_UNSUPPORTED;
    bool whole_numbers = beta != nullptr;
    for (int j = 0; j < 16; ++j) whole_numbers &= cb.c[j] == (float)j;
    const int form = regrouped ? REGROUPED : whole_numbers ? INT4 : TABLE;
    const int splits = w4_mid_call_splits(d_out, d_in, T, form == TABLE), steps = d_in / kBlock;
    if (splits > 1 && !part) return QBLORA_ERR_WORKSPACE;
    MidDesc d{codes, scales, beta, cb, tiled, d_out, d_in, X, T, Y, part, splits, (steps + splits - 1) / splits};
    const unsigned blocks = (unsigned)(((d_out + kMidRows - 1) / kMidRows) * splits);
    int rc;
    switch (token_blocks(T)) {
        case 1: rc = launch_tb<1>(d, blocks, st, form, block_rows, block_cols); break;
        case 2: rc = launch_tb<2>(d, blocks, st, form, block_rows, block_cols); break;
        case 3: rc = launch_tb<3>(d, blocks, st, form, block_rows, block_cols); break;
        case 4: rc = launch_tb<4>(d, blocks, st, form, block_rows, block_cols); break;
        case 5: rc = launch_tb<5>(d, blocks, st, form, block_rows, block_cols); break;
        case 6: rc = launch_tb<6>(d, blocks, st, form, block_rows, block_cols); break;
        case 7: rc = launch_tb<7>(d, blocks, st, form, block_rows, block_cols); break;
        default: rc = launch_tb<8>(d, blocks, st, form, block_rows, block_cols); break;
    }
    if (rc || splits == 1) return rc;
    const int64_t count = (int64_t)T * d_out;
    hipLaunchKernelGGL(k_w4_mid_reduce, dim3((unsigned)((count + 1023) / 1024)), dim3(256), 0, st, part, splits, count, Y);
    return launch_status();
}

}  // namespace qblora
