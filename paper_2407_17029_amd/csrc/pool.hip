// Launches of the row poolings of pool.h, and interval sampling.
#include "pool.h"

namespace qblora {

namespace {

template <int LAM_A, int LAM_B>
__global__ __launch_bounds__(256) void k_pool_rows8(PoolPair p) {
    const bool second = blockIdx.x >= p.n_a;
    const PoolDesc& d = second ? p.b : p.a;
    const int64_t c = (int64_t)(blockIdx.x - (second ? p.n_a : 0)) * 256 + threadIdx.x;       // output chunk (8 values)
    if (c >= (second ? p.chunks_b : p.chunks_a)) return;
    const uint4* in = reinterpret_cast<const uint4*>(d.in);
    uint4* out = reinterpret_cast<uint4*>(d.out);
    uint4* out_lo = reinterpret_cast<uint4*>(d.out_lo);
    if (LAM_A == LAM_B || !second) pool_chunk<LAM_A>(in, c, d.scale, out, out_lo);
    else pool_chunk<LAM_B>(in, c, d.scale, out, out_lo);
}

__global__ __launch_bounds__(256) void k_pool_rows1(const uint16_t* __restrict__ in, int64_t n_out, int lam,
                                                    float scale, uint16_t* __restrict__ out,
                                                    uint16_t* __restrict__ out_lo) {
    const int64_t o = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (o >= n_out) return;
    float acc = 0.0f;
    for (int i = 0; i < lam; ++i) acc += bf16_bits_to_float(in[o * lam + i]);
    const float v = acc * scale;
    const uint32_t h = pack_bf16(v, 0.0f) & 0xffffu;
    out[o] = (uint16_t)h;
    if (out_lo) out_lo[o] = (uint16_t)(pack_bf16(v - bf16_bits_to_float(h), 0.0f) & 0xffffu);
}

// Interval sampling (the "interval_sampling" compress operator of the ablation, Sec. 4.3):
// out[t, c] = in[t, lam*c]; 8 outputs (one 16-byte store) per thread when rows are whole chunks.
__global__ __launch_bounds__(256) void k_sample_rows(const uint16_t* __restrict__ in, int64_t T, int d, int lam,
                                                     uint16_t* __restrict__ out) {
    const int dq = d / lam;
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;   // first of 8 consecutive outputs
    const int64_t total = T * dq;
    if (i >= total) return;
    if ((dq & 7) == 0 && (reinterpret_cast<uintptr_t>(out) & 15) == 0) {
        const int64_t t = i / dq;
        const int c = (int)(i - t * dq);
        const uint16_t* src = in + t * d + (int64_t)c * lam;
        uint32_t w[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = (uint32_t)src[(2 * q) * lam] | ((uint32_t)src[(2 * q + 1) * lam] << 16);
        *reinterpret_cast<uint4*>(out + i) = make_uint4(w[0], w[1], w[2], w[3]);
        return;
    }
    for (int64_t j = i; j < i + 8 && j < total; ++j) {
        const int64_t t = j / dq;
        out[j] = in[t * d + (j - t * dq) * lam];
    }
}

}  // namespace

namespace {

template <int LAM_A>
void launch_chunks(const PoolPair& p, unsigned blocks, int lam_b, hipStream_t st) {
    switch (lam_b) {
        case 1: hipLaunchKernelGGL((k_pool_rows8<LAM_A, 1>), dim3(blocks), dim3(256), 0, st, p); break;
        case 2: hipLaunchKernelGGL((k_pool_rows8<LAM_A, 2>), dim3(blocks), dim3(256), 0, st, p); break;
        case 4: hipLaunchKernelGGL((k_pool_rows8<LAM_A, 4>), dim3(blocks), dim3(256), 0, st, p); break;
        default: hipLaunchKernelGGL((k_pool_rows8<LAM_A, 8>), dim3(blocks), dim3(256), 0, st, p); break;
    }
}

}  // namespace

int launch_pool_rows(const PoolDesc& a, const PoolDesc* b, hipStream_t st) {
    if (pool_outputs(a) <= 0) return b ? launch_pool_rows(*b, nullptr, st) : QBLORA_OK;
    if (b && (pool_outputs(*b) <= 0 || !pool_in_chunks(a) || !pool_in_chunks(*b) || (int64_t)pool_blocks(a) + pool_blocks(*b) > 0x7fffffff)) {
        const int rc = launch_pool_rows(a, nullptr, st);
        return rc ? rc : launch_pool_rows(*b, nullptr, st);
    }
    if (pool_in_chunks(a)) {
        PoolPair p{};
        p.a = a; p.n_a = pool_blocks(a); p.chunks_a = pool_outputs(a) / 8;
        if (b) { p.b = *b; p.chunks_b = pool_outputs(*b) / 8; }
        const unsigned blocks = p.n_a + (b ? pool_blocks(*b) : 0);
        const int lam_b = b ? b->lam : a.lam;
        switch (a.lam) {
            case 1: launch_chunks<1>(p, blocks, lam_b, st); break;
            case 2: launch_chunks<2>(p, blocks, lam_b, st); break;
            case 4: launch_chunks<4>(p, blocks, lam_b, st); break;
            default: launch_chunks<8>(p, blocks, lam_b, st); break;
        }
        return launch_status();
    }
    hipLaunchKernelGGL(k_pool_rows1, dim3((unsigned)((pool_outputs(a) + 255) / 256)), dim3(256), 0, st,
                       reinterpret_cast<const uint16_t*>(a.in), pool_outputs(a), a.lam, a.scale, reinterpret_cast<uint16_t*>(a.out),
                       reinterpret_cast<uint16_t*>(a.out_lo));
    return launch_status();
}

int launch_sample_rows(const qblora_bf16* in, int64_t T, int d, int lam, qblora_bf16* out, hipStream_t st) {
    if (T <= 0 || d <= 0 || lam <= 0 || d % lam != 0) return QBLORA_ERR_SHAPE;
    const int64_t total = T * (d / lam);
    hipLaunchKernelGGL(k_sample_rows, dim3((unsigned)((total + 2047) / 2048)), dim3(256), 0, st,
                       reinterpret_cast<const uint16_t*>(in), T, d, lam, reinterpret_cast<uint16_t*>(out));
    return launch_status();
}

}  // namespace qblora
