// Row pooling for the single-matrix adapter (QA-BLoRA, Sec. 3.3, Alg. 2): the compressed input
// AvgPool_lambda1(X) and the compressed output gradient sum_lambda2(dY) are materialised once per call
// as bf16 operands of the K-extension of the dequantize-and-contract kernel and of the dH contraction,
//
//   out[t, m] = bf16( scale * sum_{i < lam} in[t, lam*m + i] )      (sum and product in fp32)
//
// and optionally the bf16 residual out_lo = bf16(value - out), which the dH contraction adds as a
// second operand part so that only one of its two operands carries a bf16 rounding.
//
// Streaming, HBM-bound: a thread produces 8 consecutive outputs (one 16-byte store) from 8*lam
// consecutive inputs (lam 16-byte loads) when rows are whole chunks, one output otherwise.
// The launches are in pool.hip and, where a forward's pooling shares one, in prep.hip.
#pragma once
#include "common.h"

namespace qblora {

template <int LAM>
__device__ __forceinline__ void pool_chunk(const uint4* __restrict__ in, int64_t c, float scale,
                                           uint4* __restrict__ out, uint4* __restrict__ out_lo) {
    uint4 v[LAM];
#pragma unroll
    for (int i = 0; i < LAM; ++i) v[i] = in[c * LAM + i];
    float x[8 * LAM];
#pragma unroll
    for (int i = 0; i < LAM; ++i) {
        const uint32_t w[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            x[8 * i + 2 * q] = bf16_bits_to_float(w[q] & 0xffffu);
            x[8 * i + 2 * q + 1] = bf16_bits_to_float(w[q] >> 16);
        }
    }
    float o[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        float acc = x[LAM * m];
#pragma unroll
        for (int i = 1; i < LAM; ++i) acc += x[LAM * m + i];
        o[m] = acc * scale;
    }
    const uint4 h = make_uint4(pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3]), pack_bf16(o[4], o[5]), pack_bf16(o[6], o[7]));
    out[c] = h;
    if (out_lo) {
        const uint32_t hw[4] = {h.x, h.y, h.z, h.w};
        uint32_t lw[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            lw[q] = pack_bf16(o[2 * q] - bf16_bits_to_float(hw[q] & 0xffffu), o[2 * q + 1] - bf16_bits_to_float(hw[q] >> 16));
        out_lo[c] = make_uint4(lw[0], lw[1], lw[2], lw[3]);
    }
}

// Two poolings in one launch: the first n_a workgroups work on `a`.  A layer's two (dY and X of a backward) take 5 us each
// alone, most of it start and tail.
struct PoolPair { PoolDesc a, b; int64_t chunks_a, chunks_b; unsigned n_a; };

inline int64_t pool_outputs(const PoolDesc& d) { return d.T * (int64_t)(d.d / d.lam); }
// whole chunks of 8 outputs: the matrix is one run of groups of lam values (rows are contiguous)
inline bool pool_in_chunks(const PoolDesc& d) {
    const uintptr_t bits = reinterpret_cast<uintptr_t>(d.in) | reinterpret_cast<uintptr_t>(d.out) | reinterpret_cast<uintptr_t>(d.out_lo);
    return (bits & 15) == 0 && pool_outputs(d) % 8 == 0 && (d.lam == 1 || d.lam == 2 || d.lam == 4 || d.lam == 8);
}
inline unsigned pool_blocks(const PoolDesc& d) { return (unsigned)((pool_outputs(d) / 8 + 255) / 256); }

}  // namespace qblora
