// Forward of a 4-bit block-quantized layer without adapter for at most 64 tokens (merged-model inference: the INT4 weights
// that the QA-BLoRA merge of Sec. 3.3 produces, or any other quantized base).
//
//   k_w4_sums, T <= 16, 64-blocks:  Y[t, n] = sum_b ( alpha * sum_{k in b} X[t, k] c^ + beta * sum_{k in b} X[t, k] ),
//                                   c^ = bf16(c[code]): scale and offset act on the block's sums
//   k_w4_rows, everything else:     Y[t, n] = sum_k X[t, k] * bf16( c[code] * alpha (+ beta) ),   (Eq. 1) the bf16 compute
//                                   weight of the training forward
//
// Bound by the way of the data into a CU.  A vector-memory instruction takes the address path 16 cycles whether its lanes
// fetch 16 bytes or 4, and four times as long when neighbouring lanes touch different lines, so fetching codes (8 bytes a
// lane), scales and offsets (4 bytes) each in the order the MFMA operands want them costs three instructions per 640 bytes:
// 15.7 of the 20 us that 22016 x 8192 took at one token.  Here the 64 lanes of a fetch take 16 bytes each from wherever the
// next 1 KB of one block of the workgroup's rows lies -- codes, then scales, then offsets, then, with few tokens, the
// activations -- and it lands in LDS in that order; operands are read from there.  Two fetches per 48 rows instead of nine.
//
// A workgroup owns 16 RG output rows and ALL tokens; its eight waves take the 64-blocks of the input dimension in turn, each
// with stages of its own, so that there is no barrier in the loop and no partial tile leaves the workgroup (slices of the
// input dimension over workgroups cost a second launch and, at 48 tokens of 11008 x 4096, 34 MB of partial sums beside 30 MB
// of model).  A stage is free as soon as its operands are in registers, so the next fetch goes out in front of the
// arithmetic; kDepth blocks per wave are in flight.  4, 12 or 16 waves: the same times.  RG: see w4_row_groups.
//
// us against the forms before (a streaming kernel up to 16 tokens, slices above), weights rotated through HBM:
//   packed INT4      22016 x 8192   1 token  22.2 -> 19.7, 16 tokens 27.4 -> 21.6, 64 tokens 48.1 -> 36.8
//                    11008 x 4096   1 token   9.8 ->  8.1, 16 tokens 12.7 ->  9.3, 48 tokens 23.0 -> 14.1
//                     4096 x 4096   1 token   6.0 ->  5.1, 17 tokens 10.9 ->  6.9, 64 tokens 14.9 -> 10.6
//   row-major        22016 x 8192   codebook, 1 token 48 -> 28, 40 tokens 63 -> 43; INT4 72 -> 36, 90 -> 48
//   8 x 8 blocks      4096 x 11008  8 tokens 13.5 -> 9.3; 22016 x 8192 28.1 -> 25.6
// An empty launch with this prologue and the sum of the waves takes 3.3 us of each.  48 tokens, 11008 x 4096: 11.5 us
// without the fetches of the tokens, 10.9 without those of the weight, 14.1 without arithmetic: what is left is the path
// into LDS.
#include "common.h"

namespace qblora {

namespace {

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kTableReplicas = 8, kPairReplicas = 16;      // two threads write a byte's
constexpr int kSumTiles = 12;                   // 16 x 16 output tiles whose partial sums cross LDS together

struct RowsDesc {
    const uint8_t* codes; const float* scales; const float* beta; Codebook cb;
    int tiled;                 // codes (and, with 64-blocks, scales and offsets) in tile order
    int d_out, d_in;
    const qblora_bf16* X; int T;
    qblora_bf16* Y;
    int row_tiles, per_xcd;
};

typedef __attribute__((ext_vector_type(2))) float f32x2;
template <int V> struct Int { static constexpr int value = V; };

__device__ __forceinline__ uint32_t lds_address(const void* p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}
// 64 lanes x 16 bytes (4 bytes) from anywhere to lds_base + 16 (4) * lane
__device__ __forceinline__ void copy16_to_lds(const void* uniform_base, uint32_t lane_offset, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_base), "v"(lane_offset), "s"(uniform_base) : "memory");
}
__device__ __forceinline__ void gather16_to_lds(const unsigned char* p, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(lds_base), "v"(p) : "memory");
}
__device__ __forceinline__ void gather4_to_lds(const unsigned char* p, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" :: "s"(lds_base), "v"(p) : "memory");
}

// Layouts of codes and block parameters: 64-blocks in row-major arrays or in the pack's tile order, 8 x 8 blocks, blocks of
// 8 rows x 4 inputs (their parameters always row-major; TILE8_ANY: not 16-byte aligned)
enum { ROW64, TILE64, TILE8, TILE8_ANY, TILE84 };

// One block (64 inputs) of a workgroup's rows in LDS: tokens, codes (32 bytes a row), scales, offsets.
// TX: token rows; up to 8 they are fetched by the lanes that the codes leave over.
template <int RG, int TX, int FORM, int TABLE>
struct Stage {
    static constexpr bool kSplit = FORM == ROW64 || FORM == TILE8_ANY;    // block parameters by 4-byte fetches
    static constexpr int kTokenChunks = TX * 8;                            // 16-byte chunks
    static constexpr int kCodeChunks = RG * 32;
    static constexpr int kParamChunks = kSplit ? 0 : RG * (FORM == TILE84 ? 8 : 4);       // of scales, and again of offsets
    static constexpr int kCopies = TX <= 8 ? 0 : TX / 8;                   // token rows, eight each
    static constexpr int kChunks = kCodeChunks + 2 * kParamChunks + (kCopies ? 0 : kTokenChunks);
    static constexpr int kGathers = (kChunks + 63) / 64;
    static constexpr int kGathers4 = kSplit ? (RG + 1) / 2 : 0;           // 16 RG scales and as many offsets, 64 a fetch
    // where they are
    static constexpr int kCodes = kCopies * 1024;
    static constexpr int kScales = kSplit ? kCodes + kGathers * 1024 : kCodes + kCodeChunks * 16;
    static constexpr int kOffsets = kScales + (kSplit ? RG * 64 : kParamChunks * 16);
    static constexpr int kTokens = kCopies ? 0 : kCodes + (kCodeChunks + 2 * kParamChunks) * 16;
    static constexpr int kBytes = kCodes + kGathers * 1024 + kGathers4 * 256;
    static constexpr int kOps = kCopies + kGathers + kGathers4;       // vector-memory operations
    // Blocks a wave has in flight: up to four, but no more than leave a CU room for a second workgroup where that takes two
    // or three.  A lone one hides neither its start nor its sum: 22016 x 4096 at 8 tokens, 3 KB a stage, 15.0 us with four
    // in flight and 13.1 with three, 16384 x 8192 at 16 tokens 18.2 and 16.4; on at most 256 workgroups both are level.
    static constexpr int kAlone = (160 * 1024 - TABLE) / (kWaves * kBytes), kPaired = (80 * 1024 - TABLE) / (kWaves * kBytes);
    static constexpr int kStages = kPaired >= 2 ? kPaired : kAlone;
    static constexpr int kDepth = kStages > 4 ? 4 : kStages;
    static_assert(kPaired < 2 || kWaves * kDepth * kBytes + TABLE <= 80 * 1024, "two workgroups on a CU");
    static_assert(kDepth >= 1 && (kDepth - 1) * kOps < 64, "LDS; six bits of the wait counter");
};

// What the lanes fetch of the wave's blocks, one after another: a source per operation and how far it moves.
template <int RG, int TX, int FORM, int TABLE>
struct Feed {
    typedef Stage<RG, TX, FORM, TABLE> S;
    const unsigned char* src[S::kGathers + S::kGathers4];
    uint32_t step[S::kGathers + S::kGathers4];
    uint32_t x_off[S::kCopies ? S::kCopies : 1];
    const unsigned char* x;
    uint32_t lds;
    int wave, blocks, count;                                              // count: blocks of this wave (<= 0: none)

    // 16-byte chunk of a token row that sits in slot p: chunk c is in (4 (c & 1) + (c >> 1)) ^ (row >> 1 & 7), so that the
    // sixteen rows of a fragment read touch every bank once
    static __device__ __forceinline__ int chunk_in(int row, int p) {
        const int v = p ^ ((row >> 1) & 7);
        return 2 * (v & 3) + (v >> 2);
    }

    __device__ __forceinline__ void init(const RowsDesc& d, int n0, int wave_, int lane, unsigned char* mine) {
        wave = wave_;
        blocks = d.d_in / kBlock;
        count = (blocks - wave + kWaves - 1) / kWaves;
        x = reinterpret_cast<const unsigned char*>(d.X);
        lds = __builtin_amdgcn_readfirstlane(lds_address(mine));
        const bool tiled = d.tiled;
        const int d_out = d.d_out, d_in = d.d_in, nb = blocks;
        auto run = [&](int n) { return tiled ? ((int64_t)(n >> 8) * nb) * 256 + (n & 255) : (int64_t)n * nb; };
        const unsigned char* const sbase = reinterpret_cast<const unsigned char*>(d.scales);
        const unsigned char* const bbase = reinterpret_cast<const unsigned char*>(d.beta ? d.beta : d.scales);
#pragma unroll
        for (int j = 0; j < S::kGathers; ++j) {
            const int c = min(64 * j + lane, S::kChunks - 1);
            if (c < S::kCodeChunks) {
                const int n = min(n0 + (c >> 1), d_out - 1);              // rows past the end are computed, never stored
                step[j] = tiled ? 256 * 32 : 32;
                src[j] = d.codes + run(n) * 32 + (c & 1) * 16;
            } else if (c < S::kCodeChunks + 2 * S::kParamChunks) {
                const int pc = S::kParamChunks ? S::kParamChunks : 1;
                const int p = (c - S::kCodeChunks) % pc;
                const unsigned char* const base = c < S::kCodeChunks + pc ? sbase : bbase;
                if constexpr (FORM == TILE84) {
                    step[j] = 64;
                    src[j] = base + ((int64_t)min((n0 >> 3) + (p >> 2), (d_out >> 3) - 1) * (d_in >> 2) + 4 * (p & 3)) * 4;
                } else if constexpr (FORM == TILE8) {
                    step[j] = 32;
                    src[j] = base + ((int64_t)min((n0 >> 3) + (p >> 1), (d_out >> 3) - 1) * (d_in >> 3) + 4 * (p & 1)) * 4;
                } else {                                                  // four rows of a tile (tiles are whole)
                    step[j] = 1024;
                    src[j] = base + run(min(n0 + 4 * p, (d_out - 1) & ~3)) * 4;
                }
            } else {
                const int p = c - S::kCodeChunks - 2 * S::kParamChunks, row = p >> 3;
                step[j] = 128;
                src[j] = x + (int64_t)min(row, d.T - 1) * d_in * 2 + chunk_in(row, p & 7) * 16;
            }
        }
#pragma unroll
        for (int j = 0; j < S::kGathers4; ++j) {                          // no offsets: the last scale again (same line)
            const int u = min(64 * j + lane, (d.beta ? 2 : 1) * 16 * RG - 1), v = u % (16 * RG);
            const unsigned char* const base = u < 16 * RG ? sbase : bbase;
            if constexpr (FORM == TILE8_ANY) {                            // value v: block row v >> 3, column v & 7
                step[S::kGathers + j] = 32;
                src[S::kGathers + j] = base + ((int64_t)min((n0 >> 3) + (v >> 3), (d_out >> 3) - 1) * (d_in >> 3) + (v & 7)) * 4;
            } else {
                step[S::kGathers + j] = 4;
                src[S::kGathers + j] = base + run(min(n0 + v, d_out - 1)) * 4;
            }
        }
#pragma unroll
        for (int j = 0; j < S::kGathers + S::kGathers4; ++j) {
            src[j] += (uint64_t)step[j] * wave;
            step[j] *= kWaves;
        }
#pragma unroll
        for (int j = 0; j < S::kCopies; ++j) {
            const int row = 8 * j + (lane >> 3);
            x_off[j] = (uint32_t)((int64_t)min(row, d.T - 1) * d_in * 2 + chunk_in(row, lane & 7) * 16);
        }
    }
    // fetches block i of the wave (i = 0, 1, 2, ... in turn, below count) into a stage
    __device__ __forceinline__ void issue(int i, int stage) {
        const uint32_t to = lds + stage * S::kBytes;
#pragma unroll
        for (int j = 0; j < S::kGathers; ++j) gather16_to_lds(src[j], to + S::kCodes + j * 1024);
#pragma unroll
        for (int j = 0; j < S::kGathers4; ++j) gather4_to_lds(src[S::kGathers + j], to + S::kScales + j * 256);
#pragma unroll
        for (int j = 0; j < S::kGathers + S::kGathers4; ++j) src[j] += step[j];
        const int64_t b = wave + i * kWaves;
#pragma unroll
        for (int j = 0; j < S::kCopies; ++j) copy16_to_lds(x + b * 128, x_off[j], to + j * 1024);
    }
    __device__ __forceinline__ void start() {
#pragma unroll
        for (int u = 0; u < S::kDepth; ++u)
            if (u < count) issue(u, u);
    }
    // Walks the wave's blocks: block(stage, refill) reads a block's operands out of its stage, has it refilled and contracts
    // them.  A block is in when only the operations of those fetched after it are outstanding; none is fetched past the end,
    // which for short rows were more than all others (1024 inputs: two blocks a wave, four ahead of each).
    template <typename Block>
    __device__ __forceinline__ void walk(Block block) {
        constexpr int D = S::kDepth;
        int i = 0, stage = 0;
        for (; i + D < count; ++i) {
            asm volatile("s_waitcnt vmcnt(%0)" :: "n"((D - 1) * S::kOps) : "memory");
            block(stage, [&]() __attribute__((always_inline)) { issue(i + D, stage); });
            stage = stage + 1 == D ? 0 : stage + 1;
        }
        auto last = [&](auto left) __attribute__((always_inline)) {
            if (count - i < left.value) return;
            asm volatile("s_waitcnt vmcnt(%0)" :: "n"((left.value - 1) * S::kOps) : "memory");
            block(stage, []() __attribute__((always_inline)) {});
            stage = stage + 1 == D ? 0 : stage + 1;
            ++i;
        };
        static_assert(D <= 4, "four calls");
        if constexpr (D > 3) last(Int<4>{});
        if constexpr (D > 2) last(Int<3>{});
        if constexpr (D > 1) last(Int<2>{});
        last(Int<1>{});
    }
};

// scale or offset of inputs 0 .. 3, 4 .. 7, 8 .. 11, 12 .. 15 of the lane's sixteen of a block, for row group g
template <int FORM>
__device__ __forceinline__ f32x4 params_of(const unsigned char* p, int g, int r, int q) {
    if constexpr (FORM == TILE84) {
        return *reinterpret_cast<const f32x4*>(p + g * 128 + (r >> 3) * 64 + q * 16);
    } else if constexpr (FORM == TILE8 || FORM == TILE8_ANY) {
        const f32x2 two = *reinterpret_cast<const f32x2*>(p + g * 64 + (r >> 3) * 32 + q * 8);
        return f32x4{two.x, two.x, two.y, two.y};
    } else {
        const float one = *reinterpret_cast<const float*>(p + g * 64 + r * 4);
        return f32x4{one, one, one, one};
    }
}

// The two code values of byte v, out of scalar registers: a lookup in the kernel's arguments would be a vector load, and its
// data are awaited behind all copies issued before it.
__device__ __forceinline__ float2 codes_of(const Codebook& cb, int v) {
    float2 e = make_float2(cb.c[0], cb.c[0]);
#pragma unroll
    for (int j = 1; j < 16; ++j) {
        e.x = (v & 15) == j ? cb.c[j] : e.x;
        e.y = (v >> 4) == j ? cb.c[j] : e.y;
    }
    return e;
}

// RG: groups of 16 output rows of a workgroup; TB: groups of 16 tokens, of which the first TX rows are there (TX <= 8:
// one group); INT: the codebook is 0, 1, ..., 15 (and tile-ordered 64-blocks have their nibbles regrouped by the pack)
template <int RG, int TX, int FORM, bool INT>
__global__ __launch_bounds__(kThreads) void k_w4_rows(RowsDesc d) {
    constexpr int TB = (TX + 15) / 16, kTable = INT ? 0 : 256 * kTableReplicas * (int)sizeof(float2);
    typedef Feed<RG, TX, FORM, kTable> F;
    typedef typename F::S S;
    extern __shared__ __align__(16) unsigned char smem[];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int r = lane & 15, q = lane >> 4;
    const int tile = (blockIdx.x & 7) * d.per_xcd + (blockIdx.x >> 3);
    if (tile >= d.row_tiles) return;
    const int n0 = tile * (16 * RG);

    unsigned char* const mine = smem + wave * S::kDepth * S::kBytes;
    F feed;
    feed.init(d, n0, wave, lane, mine);
    feed.start();
    float2* const sT = reinterpret_cast<float2*>(smem + kWaves * S::kDepth * S::kBytes);
    if constexpr (!INT) {                                                 // while the first blocks are on their way
        const float2 e = codes_of(d.cb, t >> 1);
        float4* const to = reinterpret_cast<float4*>(sT) + t * (kTableReplicas / 4);
#pragma unroll
        for (int u = 0; u < kTableReplicas / 4; ++u) to[u] = make_float4(e.x, e.y, e.x, e.y);
        __syncthreads();
    }
    const float2* const my_table = sT + (lane & (kTableReplicas - 1));
    const int row = r & (TX - 1 < 15 ? TX - 1 : 15);                      // tokens past the end: any row (never stored)
    const int f_off = row * 128 + ((q ^ (row >> 1)) << 4);

    // the MFMA operand of one code dword: 8 inputs of the lane's row
    auto operand = [&](uint32_t cw, float a0, float a1, float b0, float b1) __attribute__((always_inline)) {
        float f[8];
        if constexpr (INT) {
            // a nibble as an E4M3 number is the code times 2^-9: two codes a conversion, exact
            const uint32_t e = cw & 0x0F0F0F0Fu, o = (cw >> 4) & 0x0F0F0F0Fu;
            const f32x2 p0 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(e, 512.0f, false);
            const f32x2 p1 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(e, 512.0f, true);
            const f32x2 p2 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(o, 512.0f, false);
            const f32x2 p3 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(o, 512.0f, true);
            if constexpr (FORM == TILE64) {              // nibbles hold inputs 0, 2, 4, 6, 1, 3, 5, 7
                f[0] = p0.x; f[4] = p0.y; f[1] = p1.x; f[5] = p1.y; f[2] = p2.x; f[6] = p2.y; f[3] = p3.x; f[7] = p3.y;
            } else {
                f[0] = p0.x; f[2] = p0.y; f[4] = p1.x; f[6] = p1.y; f[1] = p2.x; f[3] = p2.y; f[5] = p3.x; f[7] = p3.y;
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float2 tv = my_table[((cw >> (8 * i)) & 0xffu) * kTableReplicas];
                f[2 * i] = tv.x; f[2 * i + 1] = tv.y;
            }
        }
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            w[i] = pack_bf16(__fmaf_rn(f[2 * i], i < 2 ? a0 : a1, i < 2 ? b0 : b1), __fmaf_rn(f[2 * i + 1], i < 2 ? a0 : a1, i < 2 ? b0 : b1));
        return __builtin_bit_cast(bf16x8, make_uint4(w[0], w[1], w[2], w[3]));
    };

    f32x4 acc[RG][TB];
#pragma unroll
    for (int g = 0; g < RG; ++g)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) acc[g][tb] = f32x4{0.f, 0.f, 0.f, 0.f};

    const bool has_beta = d.beta != nullptr;
    feed.walk([&](int stage, auto refill) __attribute__((always_inline)) {
        const unsigned char* const in = mine + stage * S::kBytes;
        bf16x8 xf[2][TB];
        uint2 cw[RG];
        f32x4 a[RG], b[RG];
#pragma unroll
        for (int g = 0; g < RG; ++g) {
            cw[g] = *reinterpret_cast<const uint2*>(in + S::kCodes + g * 512 + r * 32 + q * 8);
            a[g] = params_of<FORM>(in + S::kScales, g, r, q);
            b[g] = params_of<FORM>(in + S::kOffsets, g, r, q);
            if (!(FORM == TILE64 && INT) && !has_beta) b[g] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) xf[m][tb] = *reinterpret_cast<const bf16x8*>(in + S::kTokens + tb * 2048 + (f_off ^ (m << 6)));
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                // all of it is in registers: the stage is free
        refill();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < RG; ++g)
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const bf16x8 wf = operand(m ? cw[g].y : cw[g].x, a[g][2 * m], a[g][2 * m + 1], b[g][2 * m], b[g][2 * m + 1]);
#pragma unroll
                for (int tb = 0; tb < TB; ++tb) acc[g][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, xf[m][tb], acc[g][tb], 0, 0, 0);
            }
    });

    // ---- the waves' sums, added in wave order: the lane holds token 16 tb + r, rows 16 g + 4 q .. + 3 ------------------
    float* const red = reinterpret_cast<float*>(smem);
    const int d_out = d.d_out;
    const bool whole = (d_out & 3) == 0 && (reinterpret_cast<uintptr_t>(d.Y) & 7) == 0;
    constexpr int kTiles = RG * TB;
#pragma unroll
    for (int c0 = 0; c0 < kTiles; c0 += kSumTiles) {
        constexpr int kChunk = kTiles < kSumTiles ? kTiles : kSumTiles;
        __syncthreads();
#pragma unroll
        for (int e = 0; e < kChunk; ++e)
            if (c0 + e < kTiles)
                *reinterpret_cast<f32x4*>(red + ((wave * kChunk + e) * 64 + lane) * 4) = acc[(c0 + e) / TB][(c0 + e) % TB];
        __syncthreads();
        for (int e = wave; e < kChunk && c0 + e < kTiles; e += kWaves) {
            const int g = (c0 + e) / TB, tb = (c0 + e) % TB;
            f32x4 s = *reinterpret_cast<const f32x4*>(red + (e * 64 + lane) * 4);
#pragma unroll
            for (int w = 1; w < kWaves; ++w) s += *reinterpret_cast<const f32x4*>(red + ((w * kChunk + e) * 64 + lane) * 4);
            const int tok = 16 * tb + r, nb = n0 + 16 * g + 4 * q;
            if (tok >= d.T || nb >= d_out) continue;
            uint16_t* p = reinterpret_cast<uint16_t*>(d.Y) + (int64_t)tok * d_out + nb;
            const uint32_t lo = pack_bf16(s[0], s[1]), hi = pack_bf16(s[2], s[3]);
            if (whole) { *reinterpret_cast<uint2*>(p) = make_uint2(lo, hi); continue; }
            p[0] = (uint16_t)(lo & 0xffffu);
            if (nb + 1 < d_out) p[1] = (uint16_t)(lo >> 16);
            if (nb + 2 < d_out) p[2] = (uint16_t)(hi & 0xffffu);
            if (nb + 3 < d_out) p[3] = (uint16_t)(hi >> 16);
        }
    }
}

// At most 16 tokens, 64-blocks: scale and offset act on the block's sums.  REGROUPED: INT4 model with regrouped nibbles.
template <int RG, int TX, int FORM, bool REGROUPED>
__global__ __launch_bounds__(kThreads) void k_w4_sums(RowsDesc d) {
    constexpr int kTable = REGROUPED ? 0 : 256 * kPairReplicas * (int)sizeof(uint32_t);
    constexpr int NE = TX < 4 ? TX : 4;                                   // sums of the lane that belong to tokens
    typedef Feed<RG, TX, FORM, kTable> F;
    typedef typename F::S S;
    extern __shared__ __align__(16) unsigned char smem[];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int r = lane & 15, q = lane >> 4;
    const int tile = (blockIdx.x & 7) * d.per_xcd + (blockIdx.x >> 3);
    if (tile >= d.row_tiles) return;
    const int n0 = tile * (16 * RG);

    unsigned char* const mine = smem + wave * S::kDepth * S::kBytes;
    F feed;
    feed.init(d, n0, wave, lane, mine);
    feed.start();
    uint32_t* const sT = reinterpret_cast<uint32_t*>(smem + kWaves * S::kDepth * S::kBytes);
    if constexpr (!REGROUPED) {                                           // while the first blocks are on their way
        const float2 c = codes_of(d.cb, t >> 1);
        const uint32_t e = pack_bf16(c.x, c.y);
        uint4* const to = reinterpret_cast<uint4*>(sT) + t * (kPairReplicas / 8);
#pragma unroll
        for (int u = 0; u < kPairReplicas / 8; ++u) to[u] = make_uint4(e, e, e, e);
        __syncthreads();
    }
    const uint32_t* const my_table = sT + (lane & (kPairReplicas - 1));
    const int row = r & (TX - 1);
    const int f_off = row * 128 + ((q ^ (row >> 1)) << 4);
    // in registers the compiler cannot see through: one and-or per operand dword (its encoding holds no two literals)
    const uint32_t nibbles = opaque_bits(0x000F000Fu), bias = opaque_bits(0x43004300u);
    auto operand = [&](uint32_t cw) __attribute__((always_inline)) {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (REGROUPED) w[i] = ((cw >> (4 * i)) & nibbles) | bias;          // 128 + code
            else w[i] = my_table[((cw >> (8 * i)) & 0xffu) * kPairReplicas];
        }
        return __builtin_bit_cast(bf16x8, make_uint4(w[0], w[1], w[2], w[3]));
    };
    const uint32_t one_pair = pack_bf16(1.0f, 1.0f);
    const bf16x8 ones = __builtin_bit_cast(bf16x8, make_uint4(one_pair, one_pair, one_pair, one_pair));

    float acc[RG][NE];
#pragma unroll
    for (int g = 0; g < RG; ++g)
#pragma unroll
        for (int e = 0; e < NE; ++e) acc[g][e] = 0.0f;

    const bool has_beta = d.beta != nullptr;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    feed.walk([&](int stage, auto refill) __attribute__((always_inline)) {
        const unsigned char* const in = mine + stage * S::kBytes;
        bf16x8 xf[2];
        uint2 cw[RG];
        float a[RG], b[RG];
#pragma unroll
        for (int g = 0; g < RG; ++g) {
            cw[g] = *reinterpret_cast<const uint2*>(in + S::kCodes + g * 512 + r * 32 + q * 8);
            a[g] = params_of<FORM>(in + S::kScales, g, r, q)[0];
            b[g] = params_of<FORM>(in + S::kOffsets, g, r, q)[0];
            if (!REGROUPED && !has_beta) b[g] = 0.0f;
        }
#pragma unroll
        for (int m = 0; m < 2; ++m) xf[m] = *reinterpret_cast<const bf16x8*>(in + S::kTokens + (f_off ^ (m << 6)));
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                // all of it is in registers: the stage is free
        refill();
        __builtin_amdgcn_sched_barrier(0);
        f32x4 xs = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[0], ones, zero, 0, 0, 0);
        xs = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[1], ones, xs, 0, 0, 0);
#pragma unroll
        for (int g = 0; g < RG; ++g) {
            f32x4 s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[0], operand(cw[g].x), zero, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[1], operand(cw[g].y), s, 0, 0, 0);
            const float bs = REGROUPED ? __fmaf_rn(-128.0f, a[g], b[g]) : b[g];
#pragma unroll
            for (int e = 0; e < NE; ++e) acc[g][e] = __fmaf_rn(bs, xs[e], __fmaf_rn(a[g], s[e], acc[g][e]));
        }
    });

    // ---- the waves' sums, added in wave order: the lane holds row 16 g + r, tokens 4 q .. + 3 ---------------------------
    float* const red = reinterpret_cast<float*>(smem);                    // [row group][wave][token of four][lane]
    __syncthreads();
#pragma unroll
    for (int g = 0; g < RG; ++g)
#pragma unroll
        for (int e = 0; e < NE; ++e) red[((g * kWaves + wave) * NE + e) * 64 + lane] = acc[g][e];
    __syncthreads();
    for (int o = t; o < RG * NE * 64; o += kThreads) {
        const int g = o / (NE * 64), e = (o >> 6) % NE, l = o & 63;
        const int tok = 4 * (l >> 4) + e, n = n0 + 16 * g + (l & 15);
        if (tok >= d.T || n >= d.d_out) continue;
        float s = red[(g * kWaves * NE + e) * 64 + l];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) s += red[((g * kWaves + w) * NE + e) * 64 + l];
        reinterpret_cast<uint16_t*>(d.Y)[(int64_t)tok * d.d_out + n] = (uint16_t)(pack_bf16(s, s) & 0xffffu);
    }
}

template <typename K>
bool set_lds(K kernel, size_t smem) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)smem) == hipSuccess;
}

template <typename S>
constexpr size_t rows_lds(int table, int sums) {
    const size_t ring = (size_t)kWaves * S::kDepth * S::kBytes + table;
    return ring > (size_t)sums ? ring : (size_t)sums;
}

template <int RG>
int launch_grid(void (*kernel)(RowsDesc), bool lds_ok, size_t smem, RowsDesc d, hipStream_t st) {
    if (!lds_ok) return QBLORA_ERR_LAUNCH;
    d.row_tiles = (d.d_out + 16 * RG - 1) / (16 * RG);
    d.per_xcd = (d.row_tiles + 7) / 8;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(8 * d.per_xcd)), dim3(kThreads), smem, st, d);
    return launch_status();
}

template <int RG, int TX, int FORM, bool INT>
int launch_rows(const RowsDesc& d, hipStream_t st) {
    constexpr int TB = (TX + 15) / 16, table = INT ? 0 : 256 * kTableReplicas * (int)sizeof(float2);
    constexpr size_t smem = rows_lds<Stage<RG, TX, FORM, table>>(table, kWaves * (RG * TB < kSumTiles ? RG * TB : kSumTiles) * 1024);
    static const bool ok = set_lds(k_w4_rows<RG, TX, FORM, INT>, smem);
    return launch_grid<RG>(k_w4_rows<RG, TX, FORM, INT>, ok, smem, d, st);
}

template <int RG, int TX, int FORM, bool REGROUPED>
int launch_sums(const RowsDesc& d, hipStream_t st) {
    constexpr int table = REGROUPED ? 0 : 256 * kPairReplicas * (int)sizeof(uint32_t);
    constexpr size_t smem = rows_lds<Stage<RG, TX, FORM, table>>(table, RG * kWaves * (TX < 4 ? TX : 4) * 256);
    static const bool ok = set_lds(k_w4_sums<RG, TX, FORM, REGROUPED>, smem);
    return launch_grid<RG>(k_w4_sums<RG, TX, FORM, REGROUPED>, ok, smem, d, st);
}

bool int_codebook(const Codebook& cb) {
    for (int j = 0; j < 16; ++j)
        if (cb.c[j] != (float)j) return false;
    return true;
}

enum Blocks { BLOCKS_ROW64, BLOCKS_TILE64, BLOCKS_REGROUPED64, BLOCKS_8X8, BLOCKS_8X8_ANY, BLOCKS_8X4 };

// (what row_groups never asks for is not built)
template <int RG, int TX, int FORM>
int launch_either(const RowsDesc& d, bool ints, hipStream_t st) {
    if (ints) return launch_rows<RG, TX, FORM, true>(d, st);
    if constexpr (RG < 6 || TX > 8) return launch_rows<RG, TX, FORM, false>(d, st);
    return QBLORA_ERR_UNSUPPORTED;
}

template <int RG, int TX>
int launch_rows_form(const RowsDesc& d, Blocks form, bool ints, hipStream_t st) {
    switch (form) {
        case BLOCKS_8X4: return launch_either<RG, TX, TILE84>(d, ints, st);
        case BLOCKS_8X8: return launch_either<RG, TX, TILE8>(d, ints, st);
        case BLOCKS_8X8_ANY:
            if constexpr (TX <= 16) return launch_either<RG, TX, TILE8_ANY>(d, ints, st);
            else return QBLORA_ERR_SHAPE;
        default: break;
    }
    if constexpr (TX > 16) {
        switch (form) {
            case BLOCKS_ROW64: return launch_either<RG, TX, ROW64>(d, ints, st);
            case BLOCKS_TILE64: return launch_rows<RG, TX, TILE64, false>(d, st);
            default: return launch_rows<RG, TX, TILE64, true>(d, st);
        }
    }
    return QBLORA_ERR_UNSUPPORTED;
}

template <int RG, int TX>
int launch_sums_form(const RowsDesc& d, Blocks form, hipStream_t st) {
    if (form == BLOCKS_REGROUPED64) return launch_sums<RG, TX, TILE64, true>(d, st);
    if constexpr (RG < 6 || TX > 8) return form == BLOCKS_ROW64 ? launch_sums<RG, TX, ROW64, false>(d, st) : launch_sums<RG, TX, TILE64, false>(d, st);
    return QBLORA_ERR_UNSUPPORTED;
}

template <int RG>
int launch_rg(const RowsDesc& d, Blocks form, hipStream_t st) {
    const bool ints = int_codebook(d.cb);
    const int T = d.T;
    if (T <= 16 && form <= BLOCKS_REGROUPED64) {
        if constexpr (RG < 6)
            if (T == 1) return launch_sums_form<RG, 1>(d, form, st);
        if (T <= 4) return launch_sums_form<RG, 4>(d, form, st);
        return T <= 8 ? launch_sums_form<RG, 8>(d, form, st) : launch_sums_form<RG, 16>(d, form, st);
    }
    if (T <= 8) return launch_rows_form<RG, 8>(d, form, ints, st);
    if (T <= 16) return launch_rows_form<RG, 16>(d, form, ints, st);
    if (T <= 32) return launch_rows_form<RG, 32>(d, form, ints, st);
    return T <= 48 ? launch_rows_form<RG, 48>(d, form, ints, st) : launch_rows_form<RG, 64>(d, form, ints, st);
}

}  // namespace

bool w4_reads_table(const Codebook& cb, int tiled, int regrouped, int block_rows, int T) {
    return block_rows != 8 && (tiled || T <= 16) ? !regrouped : !int_codebook(cb);
}

// Row groups of a workgroup: the fewest rows on the fullest CU, rounds of 256 workgroups times the rows of one, and of equal
// ones the fewest rounds, since every round starts, fetches its tokens and sums once.  us of 1 / 2 / 3 / 4 / 6 groups, packed
// INT4: 11008 x 4096 at 48 tokens 20.4 / 16.9 / 11.4 / 12.8 / 16.9 (3: 230 workgroups), 4096 x 4096 8.5 / 9.3 / 10.2 / 11.8 /
// 16.5, 22016 x 8192 at 64 tokens 104 / 63 / 48 / 52 / 39.  What departs from it, up to 16 tokens:
//   six groups, one workgroup on a CU, are behind on short rows (22016 rows at 8 tokens: 1024 inputs 7.4 / 6.7 / 6.0 / 6.5 / 6.6,
//   4096 14.1 / 13.0 / 12.4 / 14.4 / 12.7, 13824 49.4 / 40.8 / 38.0 / 43.4 / 35.3), at one token (level: 22016 x 8192 22.8 / 22.3 /
//   22.7 / 26.6 / 22.1) and, up to 8 tokens, beside a table in LDS (codebook 22016 x 8192 29.3 / 26.1 / 24.4 / 32.1 / 26.9);
//   at one token many small workgroups hide the table (codebook 19200 x 4096 12.7 / 15.0 / 14.4 / 17.4 / 14.6; row-major 22016 x
//   8192 28.4 / 32.3 / 35.5 / 43.9 / 36.3), unless rows are short (16384 x 1024 5.2 / 4.9 / 5.4 / 4.7 / 5.8).
int w4_row_groups(int d_out, int d_in, int T, bool table) {
    int groups = 1, best = 0;
    for (const int c : {1, 2, 3, 4, 6}) {
        if (c == 6 && T <= 16 && (T == 1 || (table ? T <= 8 : d_in <= 4096))) break;
        const bool small = table && T == 1 && d_in > 2048;
        const int cost = (((d_out + 16 * c - 1) / (16 * c) + 255) / 256) * (2 * c + (small ? 0 : 1));
        if (best == 0 || cost < best) { groups = c; best = cost; }
    }
    return groups;
}

// Whether this form is the faster one.  A workgroup fetches all tokens for its rows, and their room in LDS is taken from the
// codes in flight: with few rows to a workgroup, many tokens and long rows the sliced form (w4mid.hip), whose workgroups have 128
// rows, is ahead, the earlier the further the weights come (from HBM, as layer after layer does; small layers that are called
// again come from the memory-side cache).  us here / there from HBM, then from the cache: INT4 4096 x 8192 at 48 tokens 16.5 /
// 15.8, 12.2 / 15.1, at 64 19.6 / 16.5, 14.4 / 16.0, 4096 x 13824 at 32 19.9 / 17.8, 14.9 / 17.0; 8192 x 13824 at 48 31.1 /
// 29.9, 22.9 / 27.7, at 64 36.3 / 31.1, 26.9 / 29.1, 8192 x 22016 at 32 39.2 / 33.7, 38.7 / 33.4.  Codebooks hide more of it
// behind their table (4096 x 13824 at 32 tokens 19.5 / 20.8, 15.6 / 20.2), but on tall layers in tile order the table itself is
// the limit, which the sliced form reads once for 32 tokens and more: 19200 x 8192 at 17 tokens 34.2 / 30.1, 33.8 / 28.1, 19200 x
// 13824 at 64 65.8 / 58.2, 66.9 / 58.3.  (Row-major codes: 19200 x 13824 at 17 tokens 71 / 69, all others ahead here.)  Of 6480
// calls on 17 to 64 tokens from HBM, about 60 are left that the sliced form would serve more than 3 % faster, 12 % at most.
bool w4_rows_applies(int d_out, int d_in, int T, bool table, bool tiled) {
    if (T > 64) return false;
    if (T <= 16) return true;
    const int groups = w4_row_groups(d_out, d_in, T, table);
    const int64_t tokens = (int64_t)(T <= 48 ? T : 64) * d_in;
    if (groups == 1) return tokens <= (table ? 510 : 420) * 1024;
    if (groups == 2) return tokens <= 680 * 1024;
    if (!(table && tiled)) return true;
    return groups == 6 && T <= 32 ? d_in < 4096 : (int64_t)groups * d_in < (T <= 32 ? 40 : 48) * 1024;
}

int launch_w4_rows(const uint8_t* codes, const float* scales, const float* beta, const Codebook& cb, int tiled, int d_out,
                   int d_in, const qblora_bf16* X, int T, qblora_bf16* Y, hipStream_t st, int block_rows, int regrouped,
                   int block_cols) {
    if (T < 1 || T > 64 || d_in % kBlock != 0 || d_out < 1) return QBLORA_ERR_SHAPE;
    if (block_rows == 8 && d_out % 8 != 0) return QBLORA_ERR_SHAPE;
    if (regrouped && !(beta && tiled)) return QBLORA_ERR_UNSUPPORTED;
    // the entry point's limits; token rows have 32-bit offsets
    const int64_t code_bytes = ((int64_t)d_out + 255) / 256 * 256 * (d_in / 2);
    if (T <= 16 && !(block_rows == 8 && block_cols == 4) && code_bytes >= (int64_t)1 << 31) return QBLORA_ERR_UNSUPPORTED;
    if (code_bytes >= (int64_t)1 << 32 || (int64_t)T * d_in * 2 >= (int64_t)1 << 32) return QBLORA_ERR_SHAPE;
    RowsDesc d{codes, scales, beta, cb, tiled, d_out, d_in, X, T, Y, 0, 0};
    const bool any = ((reinterpret_cast<uintptr_t>(scales) | reinterpret_cast<uintptr_t>(beta)) & 15) != 0;
    const Blocks form = block_rows == 8 ? (block_cols == 4 ? BLOCKS_8X4 : any ? BLOCKS_8X8_ANY : BLOCKS_8X8)
                        : regrouped ? BLOCKS_REGROUPED64 : tiled ? BLOCKS_TILE64 : BLOCKS_ROW64;
    switch (w4_row_groups(d_out, d_in, T, w4_reads_table(cb, tiled, regrouped, block_rows, T))) {
        case 1: return launch_rg<1>(d, form, st);
        case 2: return launch_rg<2>(d, form, st);
        case 3: return launch_rg<3>(d, form, st);
        case 4: return launch_rg<4>(d, form, st);
        default: return launch_rg<6>(d, form, st);
    }
}

}  // namespace qblora
