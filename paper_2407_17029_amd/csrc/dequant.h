// The weight dequantized once, as the operand of the contraction in dense.hip: what one workgroup of 256 threads does.
// The pass shares its launches with small kernels that neither wait for it nor delay it (the adapter's re-layouts in
// prep.hip, the gradients' reduction in grads.hip): those take 4 to 9 us of which most is latency.
#pragma once
#include <type_traits>

#include "common.h"

namespace qblora {

constexpr int kDequantLds = 64 * 256 + 64;
struct __align__(16) DequantLds { unsigned char tile[64 * 256]; float lut[16]; };
static_assert(sizeof(DequantLds) == kDequantLds, "LDS of a workgroup");

__device__ __forceinline__ float group_scale(const DequantDesc& d, int64_t blk) {     // = grouped_scale()
    const int64_t g = d.scale_group == 256 ? blk >> 8 : blk / d.scale_group;
    return __fmaf_rn(e4m3_to_float(d.scale_codes[blk]), d.scale_step[g], d.scale_mid[g]);
}

// The bf16 compute weight in MFMA operand order (see DequantDesc): the weight itself.
// A workgroup owns 64 stored rows x 128 inputs.  A thread dequantizes 32 inputs of one stored row (16 bytes of
// codes; four lanes read 64 contiguous bytes of a row) into four 16-byte chunks of an LDS tile [n][16 chunks], chunk
// c of row n at position c ^ (n & 15); operand order only regroups whole chunks -- lane l = r + 16*g of the k slice
// j takes chunk 4j + g of row r -- so each wave reads its pieces back with 16-byte LDS loads (16 consecutive rows of
// one chunk lie in 16 different positions) and stores 1 KB per instruction, 4 KB contiguous per wave.  (The first form
// let a lane load the 32 code bytes of its row's block, twice per row: both lanes of a row need every other dword;
// it streamed at 0.60 of the HBM peak.)
// BETA: offsets present; GEOM: block shape, and grouped scales reconstructed here -- compile-time, so that
// a launch carries neither the other geometries' loads nor both of multiply and multiply-add with a select per weight
// (380 -> 230 vector instructions per thread).
template <bool BETA, int GEOM>
__device__ __forceinline__ void dequantize_block(const DequantDesc& d, const unsigned bid, DequantLds& s) {
    constexpr int block_rows = GEOM == EIGHT_BY_8 || GEOM == EIGHT_BY_4 ? 8 : 1, block_cols = GEOM == EIGHT_BY_4 ? 4 : 8;
    const uint8_t* __restrict__ const codes = d.codes;
    const float* __restrict__ const scales = d.scales;
    const float* __restrict__ const beta = d.beta;
    uint4* __restrict__ const out = d.out;
    const int d_out = d.d_out, d_in = d.d_in;
    float (&lut)[16] = s.lut;
    uint4 (*const tile)[16] = reinterpret_cast<uint4 (*)[16]>(s.tile);     // [n][chunk of 8 k], positions swizzled
    const int t = threadIdx.x;
    if (t < 16) lut[t] = d.cb.c[t];
    __syncthreads();
    const int n_tiles = d_out / 64;                              // d_out is a multiple of 64 here
    const int kt = bid / n_tiles;                               // 128 inputs
    const int nt = bid % n_tiles;                               // 64 stored rows
    {
        const int row = t >> 2, piece = t & 3;                  // stored row in tile, 32 inputs
        const int64_t n = (int64_t)nt * 64 + row;
        const int k0 = kt * 128 + piece * 32;
        u32x4_any cq = {0u, 0u, 0u, 0u};
        float a1 = 0.0f, b1 = 0.0f;
        float4 a4 = make_float4(0.f, 0.f, 0.f, 0.f), b4 = make_float4(0.f, 0.f, 0.f, 0.f), a4b = a4, b4b = b4;
        if (k0 < d_in) {                                        // d_in % 64 == 0: the last tile may be half
            cq = *reinterpret_cast<const u32x4_any*>(codes + n * (d_in / 2) + k0 / 2);
            if constexpr (block_rows == 8 && block_cols == 4) {  // eight block columns of 4 inputs
                const int64_t blk = (n >> 3) * (int64_t)(d_in / 4) + k0 / 4;
                a4 = *reinterpret_cast<const float4*>(scales + blk);
                a4b = *reinterpret_cast<const float4*>(scales + blk + 4);
                if constexpr (BETA) { b4 = *reinterpret_cast<const float4*>(beta + blk); b4b = *reinterpret_cast<const float4*>(beta + blk + 4); }
            } else if constexpr (block_rows == 8) {              // four block columns of 8 inputs
                const int64_t blk = (n >> 3) * (int64_t)(d_in / 8) + k0 / 8;
                a4 = *reinterpret_cast<const float4*>(scales + blk);
                if constexpr (BETA) b4 = *reinterpret_cast<const float4*>(beta + blk);
            } else {
                const int64_t blk = n * (int64_t)(d_in / kBlock) + k0 / kBlock;
                a1 = GEOM == ROWS_GROUPED ? group_scale(d, blk) : scales[blk];
                if constexpr (BETA) b1 = beta[blk];
            }
        }
        const uint32_t cw[4] = {cq.x, cq.y, cq.z, cq.w};
        const float as[8] = {a4.x, a4.y, a4.z, a4.w, a4b.x, a4b.y, a4b.z, a4b.w};
        const float bs[8] = {b4.x, b4.y, b4.z, b4.w, b4b.x, b4b.y, b4b.z, b4b.w};
        constexpr bool half = block_rows == 8 && block_cols == 4;   // two blocks per chunk of 8 inputs
#pragma unroll
        for (int c = 0; c < 4; ++c) {                           // chunk 4*piece + c: 8 inputs
            const float a = half ? as[2 * c] : block_rows == 8 ? as[c] : a1, be = half ? bs[2 * c] : block_rows == 8 ? bs[c] : b1;
            const float a_hi = half ? as[2 * c + 1] : a, be_hi = half ? bs[2 * c + 1] : be;    // inputs 4 .. 7 of the chunk
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float cv = lut[(cw[c] >> (4 * j)) & 15];
                v[j] = BETA ? __fmaf_rn(cv, j < 4 ? a : a_hi, j < 4 ? be : be_hi) : __fmul_rn(cv, j < 4 ? a : a_hi);
            }
            tile[row][(4 * piece + c) ^ (row & 15)] =
                make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]));
        }
    }
    __syncthreads();
    {
        const int w = t >> 6, lane = t & 63, row = 16 * w + (lane & 15), g = lane >> 4;
        const int64_t rb = (int64_t)nt * 4 + w;                 // 16-row block of the weight
        if (rb * 16 < d_out) {
            const int64_t kb_count = d_in / 32;                 // 32-wide k slices of a row block
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t js = (int64_t)kt * 4 + q;
                const uint4 o = tile[row][(4 * q + g) ^ (row & 15)];
                if (js < kb_count) out[(rb * kb_count + js) * 64 + lane] = o;
            }
        }
    }
}

// The same for the transposed weight (operand rows = inputs k, contraction = stored rows n), which the
// backward contraction reads.  A workgroup owns 64 stored rows x 128 inputs.  A thread dequantizes 32 inputs of
// one stored row (16 bytes of codes; four lanes read 64 contiguous bytes of a row) and writes them as four
// 16-byte chunks into an LDS tile in the stored orientation, [n][128 k] with 256-byte rows; the transposition is
// left to the transposing LDS read ds_read_b64_tr_b16 (a group of 16 lanes that points at 4 rows x 16 columns
// gets, lane i, column i of the four rows): two of them give a lane the 8 consecutive n of its k that the
// operand order wants.  Logical chunk c of row n sits at chunk position c ^ ((n & 3) << 2) ^ ((n & 8) >> 2), so that
// the four rows of a transposing read, and those of the neighbouring lane group eight rows on, lie in different
// banks.  Each wave then stores 1 KB pieces (lane l = r + 16*g holds k = r, n = 8g .. + 7 of the slice).  (The first form read 4 bytes of codes per thread and wrote 2-byte elements
// into a [k][n] tile: 57 % of its LDS cycles were bank conflicts and it streamed at 0.49 of the HBM peak.)
typedef __attribute__((ext_vector_type(4))) short s16x4_t;
template <bool BETA, int GEOM>
__device__ __forceinline__ void dequantize_t_block(const DequantDesc& d, const unsigned bid, DequantLds& s) {
    constexpr int block_rows = GEOM == EIGHT_BY_8 || GEOM == EIGHT_BY_4 ? 8 : 1, block_cols = GEOM == EIGHT_BY_4 ? 4 : 8;
    const uint8_t* __restrict__ const codes = d.codes;
    const float* __restrict__ const scales = d.scales;
    const float* __restrict__ const beta = d.beta;
    uint4* __restrict__ const out = d.out;
    const int d_out = d.d_out, d_in = d.d_in;
    float (&lut)[16] = s.lut;
    unsigned char* const tile = s.tile;                          // [n][128 k] bf16, chunks swizzled
    const int t = threadIdx.x;
    if (t < 16) lut[t] = d.cb.c[t];
    __syncthreads();
    const int n_tiles = d_out / 64;                             // d_out is a multiple of 64 here
    const int kt = bid / n_tiles;                               // 128 inputs
    const int nt = bid % n_tiles;                               // 64 stored rows
    {
        const int row = t >> 2, piece = t & 3;                  // stored row in tile, 32 inputs
        const int64_t n = (int64_t)nt * 64 + row;
        const int k0 = kt * 128 + piece * 32;
        u32x4_any cq = {0u, 0u, 0u, 0u};
        float a1 = 0.0f, b1 = 0.0f;
        float4 a4 = make_float4(0.f, 0.f, 0.f, 0.f), b4 = make_float4(0.f, 0.f, 0.f, 0.f), a4b = a4, b4b = b4;
        if (k0 < d_in) {                                        // d_in % 64 == 0: the last tile may be half
            cq = *reinterpret_cast<const u32x4_any*>(codes + n * (d_in / 2) + k0 / 2);
            if constexpr (block_rows == 8 && block_cols == 4) {  // eight block columns of 4 inputs
                const int64_t blk = (n >> 3) * (int64_t)(d_in / 4) + k0 / 4;
                a4 = *reinterpret_cast<const float4*>(scales + blk);
                a4b = *reinterpret_cast<const float4*>(scales + blk + 4);
                if constexpr (BETA) { b4 = *reinterpret_cast<const float4*>(beta + blk); b4b = *reinterpret_cast<const float4*>(beta + blk + 4); }
            } else if constexpr (block_rows == 8) {              // four block columns of 8 inputs
                const int64_t blk = (n >> 3) * (int64_t)(d_in / 8) + k0 / 8;
                a4 = *reinterpret_cast<const float4*>(scales + blk);
                if constexpr (BETA) b4 = *reinterpret_cast<const float4*>(beta + blk);
            } else {
                const int64_t blk = n * (int64_t)(d_in / kBlock) + k0 / kBlock;
                a1 = GEOM == ROWS_GROUPED ? group_scale(d, blk) : scales[blk];
                if constexpr (BETA) b1 = beta[blk];
            }
        }
        const uint32_t cw[4] = {cq.x, cq.y, cq.z, cq.w};
        const float as[8] = {a4.x, a4.y, a4.z, a4.w, a4b.x, a4b.y, a4b.z, a4b.w};
        const float bs[8] = {b4.x, b4.y, b4.z, b4.w, b4b.x, b4b.y, b4b.z, b4b.w};
        constexpr bool half = block_rows == 8 && block_cols == 4;   // two blocks per chunk of 8 inputs
#pragma unroll
        for (int c = 0; c < 4; ++c) {                           // chunk 4*piece + c: 8 inputs
            const float a = half ? as[2 * c] : block_rows == 8 ? as[c] : a1, be = half ? bs[2 * c] : block_rows == 8 ? bs[c] : b1;
            const float a_hi = half ? as[2 * c + 1] : a, be_hi = half ? bs[2 * c + 1] : be;    // inputs 4 .. 7 of the chunk
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float cv = lut[(cw[c] >> (4 * j)) & 15];
                v[j] = BETA ? __fmaf_rn(cv, j < 4 ? a : a_hi, j < 4 ? be : be_hi) : __fmul_rn(cv, j < 4 ? a : a_hi);
            }
            const int pos = (4 * piece + c) ^ ((row & 3) << 2) ^ ((row & 8) >> 2);
            *reinterpret_cast<uint4*>(tile + row * 256 + pos * 16) =
                make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]));
        }
    }
    __syncthreads();
    {
        const int w = t >> 6, lane = t & 63, g = lane >> 4, sl = lane & 15;
        const int s = w >> 1;                                   // 32 stored rows of the tile
        const int frow = 8 * g + (sl >> 2);                     // row inside the 32-row slice this lane points at
        const int64_t kb_count = d_out / 32;                    // slices of the contraction (stored rows)
#pragma unroll
        for (int q = 0; q < 4; ++q) {                           // 16 inputs each
            const int kb = 4 * (w & 1) + q, col = 16 * kb + 4 * (sl & 3);
            const unsigned char* p = tile + (32 * s + frow) * 256 +
                                     ((((col >> 3) ^ ((frow & 3) << 2) ^ ((frow & 8) >> 2)) & 15) << 4) + ((col >> 2) & 1) * 8;
            const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(p));
            const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(p + 4 * 256));
            const int64_t kb16 = (int64_t)kt * 8 + kb;
            if (kb16 * 16 < d_in) {
                uint4 o;
                o.x = __builtin_bit_cast(uint2, lo).x; o.y = __builtin_bit_cast(uint2, lo).y;
                o.z = __builtin_bit_cast(uint2, hi).x; o.w = __builtin_bit_cast(uint2, hi).y;
                out[(kb16 * kb_count + (int64_t)nt * 2 + s) * 64 + lane] = o;
            }
        }
    }
}

// f(offsets present, block geometry) with compile-time arguments
template <typename F>
inline void with_form(const DequantDesc& d, F f) {
    auto geom = [&](auto beta) {
        switch (d.geom) {
            case ROWS: f(beta, std::integral_constant<int, ROWS>{}); break;
            case EIGHT_BY_8: f(beta, std::integral_constant<int, EIGHT_BY_8>{}); break;
            case EIGHT_BY_4: f(beta, std::integral_constant<int, EIGHT_BY_4>{}); break;
            default: f(beta, std::integral_constant<int, ROWS_GROUPED>{});
        }
    };
    if (d.beta) geom(std::true_type{}); else geom(std::false_type{});
}

}  // namespace qblora
