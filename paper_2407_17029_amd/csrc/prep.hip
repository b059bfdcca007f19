// Launches of the re-layouts of prep.h, alone or with the weight of a call that dequantizes it once, and the operands of the
// alternative scale operators.
#include "dequant.h"
#include "pool.h"
#include "prep.h"

namespace qblora {

namespace {

__global__ __launch_bounds__(256) void k_adapter_prep(PrepDesc d) {
    __shared__ __align__(16) unsigned char lds[kPrepLds];
    prep_block(d, blockIdx.x, lds);
}

// The re-layouts and, behind them, the weight itself in one launch: both are done before the narrow GEMM and the
// contraction that wait for them, and the few workgroups of the first cost no launch of their own (4 to 5 us).
template <bool BETA, int GEOM>
__global__ __launch_bounds__(256) void k_prep_dequantize(PrepDesc p, DequantDesc q) {
    __shared__ __align__(16) unsigned char lds[kPrepLds > kDequantLds ? kPrepLds : kDequantLds];
    const int n = p.blocks();
    if ((int)blockIdx.x < n) prep_block(p, blockIdx.x, lds);
    else dequantize_block<BETA, GEOM>(q, blockIdx.x - n, *reinterpret_cast<DequantLds*>(lds));
}

// The same with the pooled input of the single-matrix adapter, which waits for nothing either: a launch of its own takes 5 us,
// most of it start and tail.  A layer's forward and backward on 1024 tokens of 4096 x 4096 109.6 -> 105.9 us, on 118 to 5065
// tokens of other shapes 1 to 6 % less, no shape more; hence one rule: whole chunks and a lambda that pool_chunk knows.
struct PoolJob { PoolDesc d; int64_t chunks; unsigned blocks; };
__device__ __forceinline__ void pool_block(const PoolJob& p, unsigned block) {
    const int64_t c = (int64_t)block * 256 + threadIdx.x;
    if (c >= p.chunks) return;
    const uint4* const in = reinterpret_cast<const uint4*>(p.d.in);
    uint4* const out = reinterpret_cast<uint4*>(p.d.out);
    switch (p.d.lam) {
        case 1: pool_chunk<1>(in, c, p.d.scale, out, nullptr); break;
        case 2: pool_chunk<2>(in, c, p.d.scale, out, nullptr); break;
        case 4: pool_chunk<4>(in, c, p.d.scale, out, nullptr); break;
        default: pool_chunk<8>(in, c, p.d.scale, out, nullptr);
    }
}
__global__ __launch_bounds__(256) void k_prep_pool(PrepDesc p, PoolJob j) {
    __shared__ __align__(16) unsigned char lds[kPrepLds];
    if (blockIdx.x < j.blocks) pool_block(j, blockIdx.x);
    else prep_block(p, blockIdx.x - j.blocks, lds);
}
template <bool BETA, int GEOM>
__global__ __launch_bounds__(256) void k_prep_pool_dequantize(PrepDesc p, PoolJob j, DequantDesc q) {
    __shared__ __align__(16) unsigned char lds[kPrepLds > kDequantLds ? kPrepLds : kDequantLds];
    const unsigned n = j.blocks + p.blocks();
    if (blockIdx.x < j.blocks) pool_block(j, blockIdx.x);
    else if (blockIdx.x < n) prep_block(p, blockIdx.x - j.blocks, lds);
    else dequantize_block<BETA, GEOM>(q, blockIdx.x - n, *reinterpret_cast<DequantLds*>(lds));
}

// Expanded adapter operand for the alternative scale operators (Sec. 4.3 "The scale operators"):
// every output element copies one source element or is zero.  Small (at most d x R elements), so one
// element per thread is enough.
struct ExpandDesc {
    const uint16_t* in; int src_rows, src_cols, transpose;
    int out_rows, out_cols, row_map, row_lam, col_map, col_lam;
    uint16_t* out;
};

__device__ __forceinline__ int map_index(int idx, int map, int lam, int n_src) {
    switch (map) {
        case MAP_DIV: return idx / lam;
        case MAP_FRONT: return idx < n_src ? idx : -1;
        case MAP_STRIDE: return idx % lam == 0 ? idx / lam : -1;
        default: return idx;
    }
}

__global__ __launch_bounds__(256) void k_expand_op(ExpandDesc d) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)d.out_rows * d.out_cols) return;
    const int r = (int)(i / d.out_cols), c = (int)(i - (int64_t)r * d.out_cols);
    const int sr = map_index(r, d.row_map, d.row_lam, d.src_rows);
    const int sc = map_index(c, d.col_map, d.col_lam, d.src_cols);
    uint16_t v = 0;
    if (sr >= 0 && sc >= 0 && sr < d.src_rows && sc < d.src_cols)
        v = d.transpose ? d.in[(int64_t)sc * d.src_rows + sr] : d.in[(int64_t)sr * d.src_cols + sc];
    d.out[i] = v;
}

}  // namespace

PrepDesc describe_prep(const qblora_bf16* A, const qblora_bf16* B, int d_in, int d_out, int R, int lam1, int lam2,
                       qblora_bf16* At_x, qblora_bf16* Bt, qblora_bf16* Bx, const ScaleTiling* sc) {
    PrepDesc d{};
    if (sc && sc->out) {
        d.scales = sc->scales; d.scale_codes = sc->scale_codes; d.scale_step = sc->scale_step; d.scale_mid = sc->scale_mid;
        d.scale_group = sc->scale_group; d.d_out = sc->d_out; d.bpr = sc->d_in / kBlock; d.scales_tiled = sc->out;
        d.nS = ((sc->d_out + 255) / 256) * ((d.bpr + 15) / 16);
    }
    if (!A || !B) At_x = Bt = Bx = nullptr;
    d.A = A; d.B = B; d.na_A = d_in / lam1; d.R = R; d.lam1 = lam1; d.cols_B = d_out / lam2; d.lam2 = lam2;
    d.At_x = At_x; d.Bt = Bt; d.Bx = Bx;
    if (At_x) { d.tilesA_a = (d.na_A + 63) / 64; d.tilesA_b = (R + 63) / 64; d.nA = d.tilesA_a * d.tilesA_b; }
    if (Bt) { d.tilesB_a = (R + 63) / 64; d.tilesB_b = (d.cols_B + 63) / 64; d.nB = d.tilesB_a * d.tilesB_b; }
    if (Bx) d.nX = (int)(((int64_t)R * d_out + 2047) / 2048);
    return d;
}

int launch_prep(const PrepDesc& d, hipStream_t st, const DequantDesc* dequant) {
    const int blocks = d.blocks();
    if (dequant) {
        if ((int64_t)blocks + dequant->blocks > 0x7fffffff) return QBLORA_ERR_UNSUPPORTED;
        ProfileScope ev(QBLORA_PROFILE_DEQUANT, st);
        with_form(*dequant, [&](auto beta, auto geom) {
            hipLaunchKernelGGL((k_prep_dequantize<beta.value, geom.value>), dim3(blocks + dequant->blocks), dim3(256), 0, st, d, *dequant);
        });
        return launch_status();
    }
    if (blocks == 0) return QBLORA_OK;
    hipLaunchKernelGGL(k_adapter_prep, dim3(blocks), dim3(256), 0, st, d);
    return launch_status();
}

int launch_prep_pool(const PrepDesc& d, const PoolDesc& pool, const DequantDesc* dequant, hipStream_t st) {
    const int64_t blocks = (int64_t)d.blocks() + (pool_outputs(pool) / 8 + 255) / 256 + (dequant ? dequant->blocks : 0);
    if (pool_outputs(pool) <= 0 || pool.out_lo || !pool_in_chunks(pool) || blocks > 0x7fffffff) {
        const int rc = launch_prep(d, st, dequant);
        return rc ? rc : launch_pool_rows(pool, nullptr, st);
    }
    const PoolJob j{pool, pool_outputs(pool) / 8, pool_blocks(pool)};
    if (dequant) {
        ProfileScope ev(QBLORA_PROFILE_DEQUANT, st);
        with_form(*dequant, [&](auto beta, auto geom) {
            hipLaunchKernelGGL((k_prep_pool_dequantize<beta.value, geom.value>), dim3((unsigned)blocks), dim3(256), 0, st, d, j, *dequant);
        });
    } else hipLaunchKernelGGL(k_prep_pool, dim3((unsigned)blocks), dim3(256), 0, st, d, j);
    return launch_status();
}

// What is refused here is refused in front of a call's first launch.
int describe_dequantize(const qblora_qweight& qw, qblora_bf16* Wop, DequantDesc* d) {
    if (qw.d_in % 64 != 0 || qw.d_out % 64 != 0 || (reinterpret_cast<uintptr_t>(Wop) & 15)) return QBLORA_ERR_UNSUPPORTED;
    if (qw.block_rows == 8 &&                             // four block parameters per 16-byte load
        ((reinterpret_cast<uintptr_t>(qw.scales) & 15) || (reinterpret_cast<uintptr_t>(qw.beta) & 15)))
        return QBLORA_ERR_UNSUPPORTED;
    const int64_t blocks = (int64_t)(qw.d_out / 64) * ((qw.d_in + 127) / 128);
    if (blocks > 0x7fffffff) return QBLORA_ERR_UNSUPPORTED;
    const bool grouped = qw.scale_mode == QBLORA_SCALES_E4M3_GROUPED;
    *d = DequantDesc{};
    d->codes = qw.codes; d->scales = qw.scales; d->beta = qw.beta;
    if (grouped) {
        d->scale_codes = qw.scale_codes; d->scale_step = qw.scale_step; d->scale_mid = qw.scale_mid; d->scale_group = qw.scale_group;
    }
    for (int j = 0; j < 16; ++j) d->cb.c[j] = qw.codebook[j];
    d->d_out = qw.d_out; d->d_in = qw.d_in; d->out = reinterpret_cast<uint4*>(Wop);
    d->geom = qw.block_rows != 8 ? (grouped ? ROWS_GROUPED : ROWS) : qw.block == 64 ? EIGHT_BY_8 : EIGHT_BY_4;
    d->blocks = (unsigned)blocks;
    return QBLORA_OK;
}

int launch_expand_op(const qblora_bf16* in, int src_rows, int src_cols, int transpose, int out_rows, int out_cols,
                     int row_map, int row_lam, int col_map, int col_lam, qblora_bf16* out, hipStream_t st) {
    if (!in || !out || src_rows <= 0 || src_cols <= 0 || out_rows <= 0 || out_cols <= 0 || row_lam <= 0 || col_lam <= 0)
        return QBLORA_ERR_SHAPE;
    ExpandDesc d{reinterpret_cast<const uint16_t*>(in), src_rows, src_cols, transpose, out_rows, out_cols,
                 row_map, row_lam, col_map, col_lam, reinterpret_cast<uint16_t*>(out)};
    const int64_t total = (int64_t)out_rows * out_cols;
    hipLaunchKernelGGL(k_expand_op, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, d);
    return launch_status();
}

}  // namespace qblora
