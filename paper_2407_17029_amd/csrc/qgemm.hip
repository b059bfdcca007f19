// Plain bf16 GEMM of the adapter path for outputs that are neither narrow (skinny.hip) nor a base contraction, and the
// dispatch of all contractions (gfx950):
//
//   C[M,N] = X2[M,K2] * W2[N/div2, K2]^T          (tile products of ragged shapes; s*U and dU of inner ranks above 512)
//
// Tiling: one workgroup of 512 threads (8 wave64) owns a BM x BN output tile and walks K in steps
// of 64.  Both operand tiles live in LDS as [row][64 k] bf16 with the
// 16-byte chunks of a row XOR-swizzled by (row ^ row>>3) & 7, double buffered, one barrier per
// step; global loads for step i+1 are issued before the MFMAs of step i.  The weight tile is the
// MFMA A operand and the token tile the B operand, so a lane ends up with 4 consecutive output
// features of one token and stores them as one 8-byte word.
#include "common.h"

namespace qblora {

namespace {

constexpr int kThreads = 512;
constexpr int kBK = 64;

__device__ __forceinline__ int swz(int row, int chunk) {
    return row * 128 + (((chunk ^ row ^ (row >> 3)) & 7) << 4);
}

template <int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(kThreads) void k_qgemm(GemmDesc d) {
    static_assert(WM * WN == 8, "8 waves");
    constexpr int TM = BM / WM, TN = BN / WN;       // wave tile: tokens x features
    constexpr int FM = TM / 32, FN = TN / 32;
    constexpr int XV = BM / 64;                      // 16-byte loads per thread for a token tile
    constexpr int WV = BN / 64;                      // ... for a plain bf16 weight tile

    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* sX = smem;                                   // 2 * BM*128 bytes
    unsigned char* sW = smem + 2 * BM * 128;                    // 2 * BN*128 bytes

    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int wm0 = (wave % WM) * TM, wn0 = (wave / WM) * TN;

    // ---- tile assignment: XCD-contiguous, grouped along tokens ---------------------------------
    const int tiles_m = (int)((d.M + BM - 1) / BM), tiles_n = (d.N + BN - 1) / BN;
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

    const int nsteps = (d.K2 + kBK - 1) / kBK;

    f32x16 acc[FN][FM];
#pragma unroll
    for (int a = 0; a < FN; ++a)
#pragma unroll
        for (int b = 0; b < FM; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.0f;

    // ---- prefetch registers ----------------------------------------------------------------------
    uint4 xr[XV];
    uint4 wr[WV];

    const int lrow = t >> 3, lchunk = t & 7;        // plain tile loader coordinates

    auto load_global = [&](int step) {
        const int k = step * kBK + lchunk * 8;
#pragma unroll
        for (int i = 0; i < XV; ++i) {
            int64_t row = m0 + lrow + 64 * i;
            if (row > d.M - 1) row = d.M - 1;
            xr[i] = (k < d.K2) ? *reinterpret_cast<const uint4*>(d.X2 + row * d.ldx2 + k) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < WV; ++i) {
            int row = n0 + lrow + 64 * i;
            if (row > d.N - 1) row = d.N - 1;
            row /= d.div2;
            wr[i] = (k < d.K2) ? *reinterpret_cast<const uint4*>(d.W2 + (int64_t)row * d.ldw2 + k) : make_uint4(0, 0, 0, 0);
        }
    };

    auto store_lds = [&](int buf) {
        unsigned char* bx = sX + buf * BM * 128;
        unsigned char* bw = sW + buf * BN * 128;
#pragma unroll
        for (int i = 0; i < XV; ++i) *reinterpret_cast<uint4*>(bx + swz(lrow + 64 * i, lchunk)) = xr[i];
#pragma unroll
        for (int i = 0; i < WV; ++i) *reinterpret_cast<uint4*>(bw + swz(lrow + 64 * i, lchunk)) = wr[i];
    };

    auto compute = [&](int buf) {
        const unsigned char* bx = sX + buf * BM * 128;
        const unsigned char* bw = sW + buf * BN * 128;
        const int r = lane & 31, hi = lane >> 5;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            bf16x8 wf[FN], xf[FM];
#pragma unroll
            for (int a = 0; a < FN; ++a)
                wf[a] = *reinterpret_cast<const bf16x8*>(bw + swz(wn0 + a * 32 + r, ks * 2 + hi));
#pragma unroll
            for (int b = 0; b < FM; ++b)
                xf[b] = *reinterpret_cast<const bf16x8*>(bx + swz(wm0 + b * 32 + r, ks * 2 + hi));
#pragma unroll
            for (int a = 0; a < FN; ++a)
#pragma unroll
                for (int b = 0; b < FM; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[a], xf[b], acc[a][b], 0, 0, 0);
        }
    };

    // ---- main loop ---------------------------------------------------------------------------------
    if (nsteps > 0) {
        load_global(0);
        store_lds(0);
        __syncthreads();
        for (int step = 0; step < nsteps; ++step) {
            const int buf = step & 1;
            const bool more = step + 1 < nsteps;
            if (more) load_global(step + 1);
            compute(buf);
            if (more) store_lds(buf ^ 1);
            __syncthreads();
        }
    }

    // ---- epilogue: lane holds features n..n+3 of one token per accumulator quad -----------------------
    const int r = lane & 31, hi = lane >> 5;
#pragma unroll
    for (int a = 0; a < FN; ++a)
#pragma unroll
        for (int b = 0; b < FM; ++b) {
            const int64_t m = m0 + wm0 + b * 32 + r;
            if (m >= d.M) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = n0 + wn0 + a * 32 + q * 8 + hi * 4;
                if (n >= d.N) continue;
                float v0 = acc[a][b][q * 4 + 0] * d.out_scale, v1 = acc[a][b][q * 4 + 1] * d.out_scale;
                float v2 = acc[a][b][q * 4 + 2] * d.out_scale, v3 = acc[a][b][q * 4 + 3] * d.out_scale;
                if (d.out_f32) {
                    *reinterpret_cast<float4*>(reinterpret_cast<float*>(d.C) + m * d.ldc + n) =
                        make_float4(v0, v1, v2, v3);
                } else {
                    uint2 o;
                    o.x = pack_bf16(v0, v1); o.y = pack_bf16(v2, v3);
                    *reinterpret_cast<uint2*>(reinterpret_cast<qblora_bf16*>(d.C) + m * d.ldc + n) = o;
                }
                if (d.C_lo) {
                    uint2 h;
                    h.x = pack_bf16(v0, v1); h.y = pack_bf16(v2, v3);
                    uint2 o;
                    o.x = pack_bf16(v0 - bf16_bits_to_float(h.x & 0xffffu), v1 - bf16_bits_to_float(h.x >> 16));
                    o.y = pack_bf16(v2 - bf16_bits_to_float(h.y & 0xffffu), v3 - bf16_bits_to_float(h.y >> 16));
                    *reinterpret_cast<uint2*>(d.C_lo + m * d.ldc + n) = o;
                }
                if (d.C2) {
                    uint2 o;
                    o.x = pack_bf16(v0 * d.c2_scale, v1 * d.c2_scale);
                    o.y = pack_bf16(v2 * d.c2_scale, v3 * d.c2_scale);
                    *reinterpret_cast<uint2*>(d.C2 + m * d.ldc + n) = o;
                }
            }
        }
}

template <int BM, int BN, int WM, int WN>
int launch_cfg(const GemmDesc& d, hipStream_t st) {
    constexpr size_t smem = 2 * (BM + BN) * 128;
    auto kern = k_qgemm<BM, BN, WM, WN>;
    // set once per instantiation; the initialisation of a function-local static is thread safe
    static const bool attr_ok = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem) == hipSuccess;
    if (!attr_ok) return QBLORA_ERR_LAUNCH;
    int64_t tiles = ((d.M + BM - 1) / BM) * ((d.N + BN - 1) / BN);
    hipLaunchKernelGGL(kern, dim3((unsigned)tiles), dim3(kThreads), smem, st, d);
    return launch_status();
}

}  // namespace

int launch_gemm(const GemmDesc& d, hipStream_t st) {
    if (d.M <= 0 || d.N <= 0) return QBLORA_OK;
    if (d.qmode == 1 || d.qmode == 4) return launch_qlinear(d, st);
    if (d.qmode == 2) return launch_few(d, st);
    if (d.qmode == 3) return launch_dense(d, st);
    if (skinny_applies(d)) return launch_skinny(d, st);
    // plain bf16 GEMMs of the adapter path that are not narrow (the tile product): 128 x 128 tiles unless
    // 256 x 256 tiles alone give every CU at least two workgroups
    const int64_t big_tiles = ((d.M + 255) / 256) * ((d.N + 255) / 256);
    if (d.N <= 128 || big_tiles < 512) return launch_cfg<128, 128, 2, 4>(d, st);
    return launch_cfg<256, 256, 2, 4>(d, st);
}

}  // namespace qblora
