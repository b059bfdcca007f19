// Forward contraction for at most 256 tokens (gfx950), straight from the 4-bit codes:
//
//   C[M,N] = X1[M,K] * Wq^T  +  X2[M,K2] * W2[N/div2, K2]^T
//
// with the compute weight of Eq. 1 (c[code]*alpha (+beta) in fp32, rounded to bf16) built in registers, bf16 MFMAs,
// fp32 accumulation; the second segment is the adapter's K-extension (qlinear.hip).
//
// The 256-token tiles of qlinear.hip leave the chip idle here: 256 tokens x 4096 features are 32 workgroups,
// and each walks all of K.  A workgroup here owns 16*TB tokens x 16*FB features and its 8 waves split K: wave w takes
// the 64-wide steps w, w + 8, ...  A lane dequantizes exactly its MFMA operand (row l & 15 of each 16-row block, 16
// consecutive k: 8 bytes of codes) through a byte-indexed pair table in LDS and loads its token operand (the same 16 k
// of 16 rows) from global memory one step ahead; no tile crosses LDS and no barrier stands in the loop.  The waves'
// partial tiles are added in wave order at the end.
//
// Bound: the address path.  Neighbouring lanes of an operand load are different rows, so a load of tokens or codes
// looks up 64 pieces of cache lines; a round of 8 steps costs 2.0 us with 32 x 32 tiles, 2.7 with 32 x 64 and 3.6 with
// 64 x 64.  us against qlinear.hip: 256 tokens 512 x 512 5.6 / 17, 4096 x 4096 34 / 60; 64 tokens 1024 x 1024
// 7.7 / 23; 200 tokens 4096 x 11008 70 / 166; 100 tokens 16384 x 8192 in 8 x 8 blocks 107 / 115.
#include "common.h"

namespace qblora {

namespace {

constexpr int kThreads = 512, kWaves = 8, kBK = 64;
constexpr int kTableBytes = 256 * 128;            // pair table: 256 entries of 8 bytes, 16 replicas

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

template <int TB, int FB, bool BETA, int BR>
struct Step {                                     // one 64-wide step of this lane
    u32x2_any cw[FB];                             // codes of 16 inputs of FB rows
    float sc[FB][BR == 8 ? 2 : 1], be[FB][BR == 8 ? 2 : 1];
    bf16x8 xf[TB][2];
};

template <int TB, int FB, bool BETA, int BR>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_few(GemmDesc d) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int BM = 16 * TB, kBN = 16 * FB, NACC = FB * TB;
    const int M = (int)d.M, N = d.N, d_in = d.d_in, K2 = d.K2, bpr = d_in / kBlock;
    const int steps1 = d_in / kBK, steps2 = (K2 + kBK - 1) / kBK;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int r = lane & 15, g = lane >> 4;

    // tiles: each XCD (workgroup id % 8) a contiguous range; the token tiles of one group of features are neighbours
    const int tiles_m = (M + BM - 1) / BM, ntiles = (int)gridDim.x;
    const int xcd = blockIdx.x & 7, q8 = ntiles >> 3, rem = ntiles & 7;
    const int L = xcd * q8 + min(xcd, rem) + (int)(blockIdx.x >> 3);
    const int m0 = (L % tiles_m) * BM, n0 = (L / tiles_m) * kBN;

    // pair table: byte b -> (c[b & 15], c[b >> 4]) at b*128 + replica*8; lane l reads replica l & 15, so the lanes of
    // a 16-lane group never collide
    if (t < 16) reinterpret_cast<float*>(smem)[t] = d.cb.c[t];
    __syncthreads();
    {
        const int b = t & 255;
        const float c_lo = reinterpret_cast<const float*>(smem)[b & 15], c_hi = reinterpret_cast<const float*>(smem)[b >> 4];
        __syncthreads();
        const float4 e = make_float4(c_lo, c_hi, c_lo, c_hi);
#pragma unroll
        for (int q = 0; q < 4; ++q) *reinterpret_cast<float4*>(smem + b * 128 + (t >> 8) * 64 + q * 16) = e;
    }
    __syncthreads();
    const unsigned char* const table = smem + r * 8;

    // lane offsets; the bases walk with the step
    uint32_t xrow = (uint32_t)r;                  // token rows past the end read the last one and are never stored
    const uint32_t last_row = (uint32_t)(M - 1 - m0), row_bytes = (uint32_t)(d.ldx1 * 2);
    const unsigned char* const xbase = reinterpret_cast<const unsigned char*>(d.X1 + (int64_t)m0 * d.ldx1);
    uint32_t coff[FB], soff[FB];
#pragma unroll
    for (int h = 0; h < FB; ++h) {
        coff[h] = (uint32_t)(16 * h + r) * (uint32_t)(d_in / 2) + 8u * g;
        soff[h] = BR == 8 ? (uint32_t)((16 * h + r) >> 3) * (uint32_t)(d_in / 8) + 2u * g : (uint32_t)(16 * h + r) * (uint32_t)bpr;
    }
    const uint8_t* const cbase = d.codes + (int64_t)n0 * (d_in / 2);
    const int64_t s0 = BR == 8 ? (int64_t)(n0 >> 3) * (d_in / 8) : (int64_t)n0 * bpr;
    const float* const sbase = d.scales + s0;
    const float* const bbase = BETA ? d.beta + s0 : nullptr;

    f32x4 acc[FB][TB];
#pragma unroll
    for (int a = 0; a < FB; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b) acc[a][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    auto load = [&](Step<TB, FB, BETA, BR>& st, int step) __attribute__((always_inline)) {
        const uint8_t* cb = cbase + (int64_t)step * 32;
        const float* sb = sbase + (int64_t)step * (BR == 8 ? 8 : 1);
        const float* bb = BETA ? bbase + (int64_t)step * (BR == 8 ? 8 : 1) : nullptr;
        const unsigned char* xb = xbase + (int64_t)step * (kBK * 2);
#pragma unroll
        for (int h = 0; h < FB; ++h) {
            st.cw[h] = *reinterpret_cast<const u32x2_any*>(cb + coff[h]);
#pragma unroll
            for (int i = 0; i < (BR == 8 ? 2 : 1); ++i) {
                st.sc[h][i] = sb[soff[h] + i];
                if constexpr (BETA) st.be[h][i] = bb[soff[h] + i];
            }
        }
        asm volatile("" : "+v"(xrow));                // the offsets are made again instead of held in TB registers
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            const uint32_t off = min(xrow + 16 * b, last_row) * row_bytes + 32u * g;
#pragma unroll
            for (int s = 0; s < 2; ++s) st.xf[b][s] = *reinterpret_cast<const bf16x8*>(xb + off + 16 * s);
        }
    };
    auto contract = [&](const Step<TB, FB, BETA, BR>& st) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            bf16x8 wf[FB];
#pragma unroll
            for (int h = 0; h < FB; ++h) {
                const uint32_t w = s ? st.cw[h].y : st.cw[h].x;
                const float sc = st.sc[h][BR == 8 ? s : 0], be = BETA ? st.be[h][BR == 8 ? s : 0] : 0.0f;
                uint32_t o[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t sh = i == 0 ? (w << 7) : (w >> (8 * i - 7));
                    const float2 c = *reinterpret_cast<const float2*>(table + (sh & 0x7f80u));
                    o[i] = BETA ? pack_bf16(__fmaf_rn(c.x, sc, be), __fmaf_rn(c.y, sc, be))
                                : pack_bf16(__fmul_rn(c.x, sc), __fmul_rn(c.y, sc));
                }
                wf[h] = __builtin_bit_cast(bf16x8, u32x4{o[0], o[1], o[2], o[3]});
            }
#pragma unroll
            for (int h = 0; h < FB; ++h)
#pragma unroll
                for (int b = 0; b < TB; ++b)
                    acc[h][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[h], st.xf[b][s], acc[h][b], 0, 0, 0);
        }
    };

    {
        Step<TB, FB, BETA, BR> p, q;
        int s = wave;
        if (s < steps1) load(p, s);
        for (; s < steps1; s += 2 * kWaves) {
            if (s + kWaves < steps1) load(q, s + kWaves);
            contract(p);
            if (s + kWaves >= steps1) break;
            if (s + 2 * kWaves < steps1) load(p, s + 2 * kWaves);
            contract(q);
        }
    }
    // K-extension: step e goes to wave (steps1 + e) % 8; chunks at or beyond K2 are zeros
    for (int e = (wave - steps1 % kWaves + kWaves) % kWaves; e < steps2; e += kWaves) {
        bf16x8 wf[FB][2], xf[TB][2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int k = e * kBK + 16 * g + 8 * s;
            const bool in = k < K2;
#pragma unroll
            for (int h = 0; h < FB; ++h) {
                const qblora_bf16* src = d.W2 + (int64_t)((uint32_t)(n0 + 16 * h + r) / (uint32_t)d.div2) * d.ldw2;
                const u32x4 v = *reinterpret_cast<const u32x4*>(src + (in ? k : 0));
                wf[h][s] = __builtin_bit_cast(bf16x8, in ? v : u32x4{0u, 0u, 0u, 0u});
            }
#pragma unroll
            for (int b = 0; b < TB; ++b) {
                const qblora_bf16* src = d.X2 + (int64_t)(m0 + min(16 * b + r, M - 1 - m0)) * d.ldx2;
                const u32x4 v = *reinterpret_cast<const u32x4*>(src + (in ? k : 0));
                xf[b][s] = __builtin_bit_cast(bf16x8, in ? v : u32x4{0u, 0u, 0u, 0u});
            }
        }
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int h = 0; h < FB; ++h)
#pragma unroll
                for (int b = 0; b < TB; ++b)
                    acc[h][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[h][s], xf[b][s], acc[h][b], 0, 0, 0);
    }

    // partial tiles through LDS, added in wave order: accumulator j of wave w at ((w*NACC + j)*64 + lane)*16
    __syncthreads();                                     // every wave is done with the table
    f32x4* const red = reinterpret_cast<f32x4*>(smem);
#pragma unroll
    for (int a = 0; a < FB; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b) red[(wave * NACC + a * TB + b) * 64 + lane] = acc[a][b];
    __syncthreads();
    qblora_bf16* const C = reinterpret_cast<qblora_bf16*>(d.C);
#pragma unroll
    for (int j0 = 0; j0 < NACC; j0 += kWaves) {
        const int j = j0 + wave;
        if (j >= NACC) break;
        f32x4 v = red[j * 64 + lane];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) v += red[(w * NACC + j) * 64 + lane];
        const int m = m0 + 16 * (j % TB) + r, n = n0 + 16 * (j / TB) + 4 * g;
        if (m < M)
            *reinterpret_cast<uint2*>(C + (int64_t)m * d.ldc + n) =
                make_uint2(pack_bf16(v[0] * d.out_scale, v[1] * d.out_scale), pack_bf16(v[2] * d.out_scale, v[3] * d.out_scale));
    }
}

template <int TB, int FB, bool BETA, int BR>
int launch_cfg(const GemmDesc& d, hipStream_t st) {
    constexpr int red = kWaves * FB * TB * 64 * 16, smem = red > kTableBytes ? red : kTableBytes;
    auto kern = k_few<TB, FB, BETA, BR>;
    // set once per instantiation; the initialisation of a function-local static is thread safe
    static const bool attr_ok = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                    hipFuncAttributeMaxDynamicSharedMemorySize, smem) == hipSuccess;
    if (!attr_ok) return QBLORA_ERR_LAUNCH;
    const int64_t tiles = ((d.M + 16 * TB - 1) / (16 * TB)) * (d.N / (16 * FB));
    hipLaunchKernelGGL(kern, dim3((unsigned)tiles), dim3(kThreads), smem, st, d);
    return launch_status();
}

template <int TB, int FB>
int launch_tile(const GemmDesc& d, hipStream_t st) {
    if (d.block_rows == 8) return d.beta ? launch_cfg<TB, FB, true, 8>(d, st) : launch_cfg<TB, FB, false, 8>(d, st);
    return d.beta ? launch_cfg<TB, FB, true, 1>(d, st) : launch_cfg<TB, FB, false, 1>(d, st);
}

}  // namespace

namespace {

// Tile (0: 32 x 32, 1: 32 x 64, 2: 64 x 64 tokens x features) by the estimated time in ns: rounds of workgroups (one per
// CU) x rounds of 8 steps x the measured time of such a round; -1 where the 256-token tiles are the faster ones.  us here /
// there: 11008 x 4096 at 128 / 160 tokens 66 / 72 and 87 / 71; 13824 x 5120 at 128 / 160 79 / 87 and 112 / 86; 22016 x 8192
// at 64 / 65 121 / 128 and 180 / 133; 8192 x 8192 at 256 tokens 121 / 123.
int few_tile(int64_t M, int N, int K) {
    static constexpr int tb[3] = {32, 32, 64}, fb[3] = {32, 64, 64}, cost[3] = {2000, 2700, 3600};
    const int64_t steps = K / kBK;
    int best = -1;
    int64_t best_t = qlinear_ns(M, N, K) + 3000;         // its longer start (512 inputs: 4 to 11 us behind)
    for (int i = 0; i < 3; ++i) {
        const int64_t wgs = ((M + tb[i] - 1) / tb[i]) * (N / fb[i]);
        const int64_t t = (wgs + 255) / 256 * ((steps + 7) / 8) * cost[i];
        if (t < best_t) { best_t = t; best = i; }
    }
    return best;
}

}  // namespace

bool few_applies(int64_t M, int N, int K) { return M <= kFewTokens && N % 64 == 0 && K % kBK == 0 && few_tile(M, N, K) >= 0; }

int launch_few(const GemmDesc& d, hipStream_t st) {
    if (d.M <= 0 || d.N <= 0) return QBLORA_OK;
    if (d.out_f32 || d.C2 || d.C_lo || !d.scales || !few_applies(d.M, d.N, d.d_in)) return QBLORA_ERR_UNSUPPORTED;
    // 8 x 8 blocks ask for block parameters on a 16-byte boundary, here as everywhere
    if (d.block_rows == 8 && ((reinterpret_cast<uintptr_t>(d.scales) & 15) || (reinterpret_cast<uintptr_t>(d.beta) & 15)))
        return QBLORA_ERR_UNSUPPORTED;
    switch (few_tile(d.M, d.N, d.d_in)) {
        case 0: return launch_tile<2, 2>(d, st);
        case 1: return launch_tile<2, 4>(d, st);
        default: return launch_tile<4, 4>(d, st);
    }
}

}  // namespace qblora
