"""Inference on at most 64 tokens (a workgroup walks the whole input dimension) at the edges of its tiles: token counts on
both sides of every form, 1, 2, 3, 4 and 6 row groups with ragged last workgroups, fewer blocks than waves."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2407_17029_amd import synth

pytestmark = pytest.mark.gpu

FORMATS = {"int4": (64, 1, True), "nf4": (64, 1, False), "8x8": (64, 8, True), "8x8_nf4": (64, 8, False), "8x4": (32, 8, True),
           "8x4_nf4": (32, 8, False)}


def _case(oracle, codebook, seed, T, d_out, d_in, fmt):
    from paper_2407_17029_amd import binding as qb
    from gpu_util import f32_to_dev, bf16_to_dev, OracleWeight
    block, rows, minmax = FORMATS[fmt]
    L = synth.make_layer(seed, T, d_out, d_in, 8, 1, 1)
    how = (qb.QUANT_MINMAX_INT4,) if minmax else (qb.QUANT_ABSMAX_CODEBOOK, codebook)
    qw = qb.qblora_quantize_blockwise(f32_to_dev(L.W), block, *how, block_rows=rows)
    ow = OracleWeight(oracle, L.W, codebook, minmax, block_rows=rows, block_cols=4 if block == 32 else 8).assert_same(qw)
    sums = T <= 16 and rows == 1                         # scale and offset act on block sums: the weight is not rounded
    ref = oracle.forward(ow.dequantize(oracle, 3 if sums else 2), L.X, None, None, 1, 1, 0.0)
    return qb, qw, bf16_to_dev(L.X), ref


@pytest.mark.parametrize("fmt", list(FORMATS))
@pytest.mark.parametrize("T,d_out,d_in", [
    (1, 8, 64), (1, 4104, 192), (2, 8200, 64), (4, 12296, 128), (5, 104, 576), (8, 16392, 64), (9, 24584, 64), (16, 40, 1024),
    (17, 4088, 192), (32, 4104, 64), (33, 8184, 64), (48, 8200, 448), (49, 12296, 64), (64, 16376, 64), (64, 16392, 128),
    (64, 72, 576), (40, 24568, 64),
    # more blocks than a wave has in flight, a ragged number of them, in every number of row groups
    (1, 4104, 2624), (2, 24584, 704), (8, 6152, 2624), (12, 18440, 1600), (16, 9224, 2368), (24, 4088, 2624), (32, 12296, 1600),
    (48, 8200, 2112), (40, 12296, 1344), (33, 16392, 1088), (64, 16376, 1600), (64, 24584, 1088), (48, 20488, 1344),
    (48, 40, 2624), (64, 72, 2624), (40, 8184, 1600), (64, 8184, 1600), (49, 11000, 1600), (64, 16392, 1216),
])
def test_edges(oracle, codebook, rules, T, d_out, d_in, fmt):
    from gpu_util import assert_close_bf16
    rows = rules.L["_ZN6qblora15w4_rows_appliesEiiibb"]
    rows.argtypes, rows.restype = [C.c_int, C.c_int, C.c_int, C.c_bool, C.c_bool], C.c_bool
    assert all(rows(d_out, d_in, T, table, tiled) for table in (False, True) for tiled in (False, True))
    print(f"case w4 rows T={T} {d_out}x{d_in} {fmt}", flush=True)
    qb, qw, X, ref = _case(oracle, codebook, 8000 + T + d_out, T, d_out, d_in, fmt)
    Y = torch.full((T + 1, d_out), 7.0, dtype=torch.bfloat16, device=X.device)
    qb.qblora_linear_decode(qw, X, Y=Y[:T])
    Yp = qb.qblora_linear_decode(qw, X, pack=qb.qblora_decode_pack(qw))
    torch.cuda.synchronize()
    assert_close_bf16(Y[:T], ref, "Y")
    assert_close_bf16(Yp, ref, "Y (packed)")
    assert torch.all(Y[T:] == 7.0)                       # nothing is written past the last token
    if fmt != "int4" or T > 16:                          # the packed INT4 sums take the 128 off in another order
        assert torch.equal(Y[:T], Yp)


@pytest.mark.parametrize("T", [3, 16])
@pytest.mark.parametrize("fmt", ["8x8", "8x8_nf4"])
def test_block_parameters_at_any_word(oracle, codebook, T, fmt):
    """Up to 16 tokens, scales and offsets of 8 x 8 blocks and Y need no more alignment than their type."""
    from gpu_util import assert_close_bf16
    d_out, d_in = 200, 320
    print(f"case w4 rows unaligned T={T} {fmt}", flush=True)
    qb, qw, X, ref = _case(oracle, codebook, 8100 + T, T, d_out, d_in, fmt)

    def moved(t):
        return None if t is None else torch.cat([t.new_zeros(1), t.reshape(-1)])[1:].view(t.shape)

    odd = qb.QWeight(d_out, d_in, qw.block, qw.codebook, qw.codes, moved(qw.scales), moved(qw.beta), block_rows=8)
    assert odd.scales.data_ptr() % 16 == 4
    Y = torch.empty(T * d_out + 1, dtype=torch.bfloat16, device=X.device)[1:].view(T, d_out)
    qb.qblora_linear_decode(odd, X, Y=Y)
    torch.cuda.synchronize()
    assert_close_bf16(Y, ref, "Y")
    assert torch.equal(Y, qb.qblora_linear_decode(qw, X))
