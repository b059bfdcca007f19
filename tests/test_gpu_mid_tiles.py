"""Inference on 65 to 256 tokens, and on fewer of few long rows: every token tile at both of its ends, one to eight slices whose
steps leave a remainder in the ring, ragged row tiles, and the three ways a code becomes a number (table, INT4, INT4 with
regrouped nibbles)."""
import ctypes as C

import pytest
import torch

from test_gpu_w4_rows import FORMATS, _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", list(FORMATS))
@pytest.mark.parametrize("T,d_out,d_in", [
    (65, 40, 64), (96, 136, 640), (97, 256, 1088), (128, 24, 2048), (129, 264, 448), (160, 8, 320), (161, 136, 192),
    (192, 128, 704), (193, 72, 2112), (224, 136, 256), (225, 40, 576), (256, 120, 832),
    (17, 40, 40000), (32, 136, 21056), (33, 264, 21504), (50, 40, 14016), (64, 72, 13760),
])
def test_token_tiles(oracle, codebook, rules, T, d_out, d_in, fmt):
    from gpu_util import assert_close_bf16
    rows = rules.L["_ZN6qblora15w4_rows_appliesEiiibb"]
    rows.argtypes, rows.restype = [C.c_int, C.c_int, C.c_int, C.c_bool, C.c_bool], C.c_bool
    assert not any(rows(d_out, d_in, T, table, True) for table in (False, True))
    print(f"case mid tiles T={T} {d_out}x{d_in} {fmt}", flush=True)
    qb, qw, X, ref = _case(oracle, codebook, 8200 + T + d_out, T, d_out, d_in, fmt)
    Y = torch.full((T + 1, d_out), 7.0, dtype=torch.bfloat16, device=X.device)
    qb.qblora_linear_decode(qw, X, Y=Y[:T])
    Yp = qb.qblora_linear_decode(qw, X, pack=qb.qblora_decode_pack(qw))
    torch.cuda.synchronize()
    assert_close_bf16(Y[:T], ref, "Y")
    assert torch.equal(Y[:T], Yp)                        # the same weight, contracted in the same order
    assert torch.all(Y[T:] == 7.0)                       # nothing is written past the last token


@pytest.mark.parametrize("fmt", list(FORMATS))
@pytest.mark.parametrize("T,d_out,d_in", [
    (161, 40, 64), (256, 264, 64), (200, 136, 128), (225, 8, 192), (256, 40, 256),          # one to four steps: fewer than the rings hold
    (192, 264, 512), (224, 128, 576),                                                   # two slices of four, of four and five
])
def test_copying_waves_on_short_slices(oracle, codebook, rules, T, d_out, d_in, fmt):
    test_token_tiles(oracle, codebook, rules, T, d_out, d_in, fmt)


@pytest.mark.parametrize("fmt", [f for f in FORMATS if "8x" not in f])
@pytest.mark.parametrize("T,d_out,d_in", [
    (161, 37, 64), (201, 130, 256), (255, 257, 448),           # one slice: odd rows, pairs of rows, one row past two tiles
    (161, 130, 2048), (201, 37, 832), (255, 257, 1088), (193, 2, 576), (256, 1, 1024),     # slices whose sums are no whole words
])
def test_copying_waves_on_odd_outputs(oracle, codebook, rules, T, d_out, d_in, fmt):
    """Outputs in 64-blocks may be any number: single stores, block parameters up to the last row, the sums' scalar path."""
    test_token_tiles(oracle, codebook, rules, T, d_out, d_in, fmt)
