"""GPU parity: dX contracted straight from the codes of the transposed weight (few tokens, wide layers), at the edges of its
two tiles, with fewer steps than the loads run ahead, every weight format and a ragged K-extension."""
import numpy as np
import pytest
import torch

from paper_2407_17029_amd import synth

pytestmark = pytest.mark.gpu

# T, d_out (contraction), d_in, R, format: tiles of 128 columns (up to 32768 columns at one token tile) and of 256
CASES = [
    (5, 64, 28160, 0, "nf4"),             # one step
    (130, 64, 24256, 8, "tile8"),         # one step and a partial extension step, half a column tile past the last whole one
    (130, 128, 20544, 0, "minmax"),
    (70, 192, 28160, 0, "grouped"),
    (1, 448, 27328, 72, "tile8_nf4"),     # the unrolled loop and its rest, two extension steps
    (257, 512, 12864, 24, "minmax"),      # two token tiles
    (1, 128, 34368, 0, "nf4"),            # 256 columns a tile, two steps
    (5, 192, 32896, 0, "tile8"),
    (130, 128, 32832, 8, "grouped"),
    (20, 320, 32832, 0, "minmax"),
    (1, 448, 36416, 24, "tile8_nf4"),
    (257, 448, 22144, 8, "nf4"),
]


def _weight(qb, oracle, codebook, W, fmt):
    from gpu_util import f32_to_dev, OracleWeight
    br = 8 if fmt.startswith("tile8") else 1
    minmax, grouped = fmt in ("minmax", "tile8"), fmt == "grouped"
    if minmax:
        qw = qb.qblora_quantize_blockwise(f32_to_dev(W), 64, qb.QUANT_MINMAX_INT4, block_rows=br)
    else:
        qw = qb.qblora_quantize_blockwise(f32_to_dev(W), 64, qb.QUANT_ABSMAX_CODEBOOK, codebook,
                                          qb.SCALES_E4M3_GROUPED if grouped else qb.SCALES_FP32, block_rows=br)
    torch.cuda.synchronize()
    return qw, OracleWeight(oracle, W, codebook, minmax, grouped, br).assert_same(qw).dequantize(oracle, 2)


@pytest.mark.parametrize("T,d_out,d_in,R,fmt", CASES)
def test_transposed_codes(rules, oracle, codebook, T, d_out, d_in, R, fmt):  # noqa: F811
    from paper_2407_17029_amd import binding as qb
    from gpu_util import bf16_to_dev, assert_close_bf16
    print(f"case transposed codes T={T} {d_out}x{d_in} R={R} {fmt}", flush=True)
    assert not rules.dense_pays_t(T, d_in, d_out, R)
    L = synth.make_layer(9100 + T + d_out, T, d_out, d_in, max(R, 8), 2, 2, b_std=0.05)
    qw, Wt = _weight(qb, oracle, codebook, L.W, fmt)
    ad = qb.Adapter(bf16_to_dev(L.A), bf16_to_dev(L.B), 2, 2, 0.5) if R else None
    A, B, s = (L.A, L.B, 0.5) if R else (None, None, 0.0)
    X, dY = bf16_to_dev(L.X), bf16_to_dev(L.dY)
    dX = torch.full((T, d_in), float("nan"), dtype=torch.bfloat16, device=X.device)
    qb.qblora_linear_bwd(qw, ad, X, dY, need_grads=False, dX=dX)
    torch.cuda.synchronize()
    assert_close_bf16(dX, oracle.backward(Wt, L.X, L.dY, A, B, 2, 2, s)[0], "dX")


@pytest.mark.parametrize("T,d_out,d_in,fmt", [(1, 192, 30528, "grouped"), (1, 448, 36416, "tile8")])
def test_single_matrix_adapter(rules, oracle, codebook, T, d_out, d_in, fmt):  # noqa: F811
    from paper_2407_17029_amd import binding as qb
    from gpu_util import bf16_to_dev, assert_close_bf16
    print(f"case transposed codes, single matrix T={T} {d_out}x{d_in} {fmt}", flush=True)
    assert not rules.dense_pays_t(T, d_in, d_out, d_out // 8)
    L = synth.make_layer(9200 + d_out, T, d_out, d_in, 8, 8, 8)
    qw, Wt = _weight(qb, oracle, codebook, L.W, fmt)
    Hb = synth.f32_to_bf16_bits(synth.normal_f32(9201, 0, (d_in // 8, d_out // 8)) * np.float32(0.02))
    dX, _ = qb.qablora_linear_bwd(qw, bf16_to_dev(Hb), 8, 8, 0.5, bf16_to_dev(L.X), bf16_to_dev(L.dY), need_dh=False)
    torch.cuda.synchronize()
    assert_close_bf16(dX, oracle.qa_backward(Wt, L.X, L.dY, Hb, 8, 8, 0.5, compute_dh=False)[0], "dX")
