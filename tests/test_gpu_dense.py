"""GPU parity: the contraction on a weight dequantized once, at the edges of its tiles and of its ring of stages."""
import numpy as np
import pytest
import torch

from paper_2407_17029_amd import synth

pytestmark = pytest.mark.gpu

# T, d_out, d_in, R: the tiles (tokens x features; forward and backward differ) follow from T and the output width, the number of
# 64-wide steps from the other width (one step up to more than the ring holds), R adds none, one partial or two steps of the
# K-extension.  Backward contractions of few output tiles are sliced, in 128 x 128 tiles here; the other tiles in slices are
# below.
CASES = [
    (4100, 4096, 64, 0),       # 192 x 192, one step; backward 128 x 128, 64 steps
    (4100, 4096, 128, 72),     # 192 x 192, two steps and a ragged extension
    (4097, 4160, 192, 8),      # 192 x 192, three steps, partial tiles on both sides
    (2048, 4096, 64, 8),       # 128 x 256, one step
    (1930, 4032, 256, 0),      # 128 x 256, partial tiles on both sides, as many steps as stages and one more
    (1270, 6528, 64, 0),       # 256 x 128, one step
    (1270, 6528, 192, 72),     # 256 x 128, three steps and a ragged extension
    (257, 64, 320, 8),         # 128 x 128, narrower than a tile
    (300, 320, 64, 24),        # 128 x 128, fewer steps than stages
    (1, 448, 128, 16),         # backward of one token; forward few
    (200, 2112, 192, 72),      # backward in slices of 128 x 128 tiles, the last one with the ragged extension; forward few
    (1000, 4160, 448, 0),      # backward in slices, no adapter, partial tiles on both sides; forward 128 x 192
    (513, 8256, 2048, 8),      # backward in slices of 128 x 128 tiles; forward 192 x 128, 64 features in the last
    (700, 8256, 1024, 8),      # forward from the codes
]


@pytest.mark.parametrize("T,d_out,d_in,R", CASES)
def test_tiles_and_stages(oracle, codebook, T, d_out, d_in, R):
    from paper_2407_17029_amd import binding as qb
    from gpu_util import f32_to_dev, bf16_to_dev, assert_close_bf16, OracleWeight
    print(f"case dense T={T} {d_out}x{d_in} R={R}", flush=True)
    # s*U enters the extension rounded to bf16 (relative 2^-9).  With B ~ N(0, 0.05^2) the adapter term is at most
    # about 0.4 rms of the output even at these short contractions, 5 * 0.4 rms at its largest element, so that
    # rounding stays below 5 * 0.4 * 2^-9 = 4e-3 rms, inside the 1e-2 bar (B ~ N(0, 0.3^2), an adapter of the
    # output's own size with peaks of 15 rms, reached 1.1e-2 from it alone).
    L = synth.make_layer(5100 + T + d_out, T, d_out, d_in, max(R, 8), 2, 2, b_std=0.05)
    qw = qb.qblora_quantize_blockwise(f32_to_dev(L.W), 64, qb.QUANT_ABSMAX_CODEBOOK, codebook)
    torch.cuda.synchronize()
    Wt = OracleWeight(oracle, L.W, codebook).assert_same(qw).dequantize(oracle, 2)
    ad = qb.Adapter(bf16_to_dev(L.A), bf16_to_dev(L.B), 2, 2, 0.5) if R else None
    A, B, s = (L.A, L.B, 0.5) if R else (None, None, 0.0)
    X, dY = bf16_to_dev(L.X), bf16_to_dev(L.dY)
    Y = torch.full((T, d_out), float("nan"), dtype=torch.bfloat16, device=X.device)
    dX = torch.full((T, d_in), float("nan"), dtype=torch.bfloat16, device=X.device)
    qb.qblora_linear_fwd(qw, ad, X, Y=Y)
    qb.qblora_linear_bwd(qw, ad, X, dY, need_grads=False, dX=dX)
    torch.cuda.synchronize()
    assert_close_bf16(Y, oracle.forward(Wt, L.X, A, B, 2, 2, s), "Y")
    assert_close_bf16(dX, oracle.backward(Wt, L.X, L.dY, A, B, 2, 2, s)[0], "dX")
    # the form that rebuilds weight tiles in LDS adds in the same order (of 1 and 200 tokens both take the one for few,
    # of 700 both take this one)
    Y2 = torch.empty_like(Y)
    qb.qblora_linear_fwd_noalloc(qw, ad, X, Y2)
    torch.cuda.synchronize()
    assert torch.equal(Y.view(torch.int16), Y2.view(torch.int16))


TILES = ["256 x 256", "128 x 256", "256 x 128", "128 x 128", "128 x 192", "192 x 128", "192 x 192"]


@pytest.mark.parametrize("T,d_out,d_in,R,tile,slices", [
    (577, 6784, 3392, 24, "128 x 256", 3),     # 65 tokens and 64 features in the last tiles; steps that do not divide evenly
    (700, 7168, 2880, 24, "256 x 128", 3),     # 188 and 64, uneven
    (257, 3904, 3648, 72, "192 x 128", 4),     # 65 and 64, uneven, a ragged extension of two steps
    (385, 4672, 2752, 72, "128 x 192", 4),     # one token past three tiles, 64, uneven
    (65, 1024, 64, 72, "128 x 128", 4),        # half a tile both ways, 18 steps
])
def test_slices_of_partial_tiles(oracle, codebook, rules, T, d_out, d_in, R, tile, slices):
    from paper_2407_17029_amd import binding as qb
    from gpu_util import f32_to_dev, bf16_to_dev, assert_close_bf16, OracleWeight
    print(f"case dense slices T={T} {d_out}x{d_in} R={R}", flush=True)
    plan = rules.dense_call_plan(T, d_in, d_out, R, 8)
    assert rules.dense_pays_t(T, d_in, d_out, R) and (TILES[plan.shape], plan.splits) == (tile, slices)
    L = synth.make_layer(5200 + T, T, d_out, d_in, max(R, 8), 2, 2, b_std=0.05)
    qw = qb.qblora_quantize_blockwise(f32_to_dev(L.W), 64, qb.QUANT_ABSMAX_CODEBOOK, codebook, tiled=False)
    Wt = OracleWeight(oracle, L.W, codebook).assert_same(qw).dequantize(oracle, 2)
    ad = qb.Adapter(bf16_to_dev(L.A), bf16_to_dev(L.B), 2, 2, 0.5) if R else None
    A, B, s = (L.A, L.B, 0.5) if R else (None, None, 0.0)
    dX = torch.full((T, d_in), float("nan"), dtype=torch.bfloat16, device="cuda")
    qb.qblora_linear_bwd(qw, ad, bf16_to_dev(L.X), bf16_to_dev(L.dY), need_grads=False, dX=dX)
    torch.cuda.synchronize()
    assert_close_bf16(dX, oracle.backward(Wt, L.X, L.dY, A, B, 2, 2, s)[0], "dX")


@pytest.mark.parametrize("T,d_out,d_in,R,tile", [
    (2049, 4480, 64, 8, "256 x 256"),       # one step and the extension; one token and half a tile past
    (8193, 1088, 64, 0, "256 x 256"),       # a single step; one token and 64 features past
    (7000, 1216, 64, 0, "256 x 256"), (7000, 1216, 192, 0, "256 x 256"),     # one and three steps; 88 tokens, 192 features in the last
    (7000, 1216, 128, 72, "256 x 256"),     # two steps and a ragged extension of two
    (1025, 5440, 64, 0, "128 x 256"),       # a single step
    (1025, 5440, 192, 72, "128 x 256"),     # as many steps as stages, and a ragged extension
    (1930, 3200, 128, 72, "256 x 128"),     # one more
    (257, 640, 64, 0, "128 x 128"),         # a single step
    (300, 640, 256, 72, "128 x 128"),       # one step more than stages
    (257, 640, 1024, 8, "128 x 128"),
    (769, 4800, 64, 0, "128 x 192"), (769, 4800, 320, 72, "128 x 192"),      # one token past; whole feature tiles
    (769, 4672, 128, 8, "128 x 192"),      # 64 features in the last tile
    (900, 4160, 64, 0, "192 x 128"), (700, 5440, 256, 72, "192 x 128"),      # partial tiles both ways
    (1153, 6592, 64, 0, "192 x 192"), (1153, 6592, 192, 72, "192 x 192"),    # one token past, 64 features in the last tile
    (577, 2112, 704, 0, "128 x 128"),       # an odd number of steps
])
def test_tiles_that_calls_take(oracle, codebook, rules, T, d_out, d_in, R, tile):
    assert TILES[rules.dense_call_plan(T, d_out, d_in, R, 1).shape] == tile
    test_tiles_and_stages(oracle, codebook, T, d_out, d_in, R)


@pytest.mark.parametrize("T,d_out,d_in,R,tile,slices", [
    (65, 2112, 320, 72, "128 x 128", 7), (129, 4096, 5504, 72, "192 x 128", 4), (65, 8192, 8384, 72, "128 x 192", 5),
    (577, 6784, 3392, 24, "128 x 256", 3), (385, 8192, 3200, 72, "256 x 128", 5), (900, 11008, 2240, 72, "192 x 192", 4),
    (385, 13248, 5824, 24, "256 x 256", 5),      # 129 tokens and 192 features in the last tiles; slices of 41 and 42 steps
])
def test_slices_that_calls_take(oracle, codebook, rules, T, d_out, d_in, R, tile, slices):
    plan = rules.dense_call_plan(T, d_in, d_out, R, 8)
    assert rules.dense_pays_t(T, d_in, d_out, R) and (TILES[plan.shape], plan.splits) == (tile, slices)
    test_tiles_and_stages(oracle, codebook, T, d_out, d_in, R)


def test_slices_with_a_single_matrix_adapter(oracle, codebook, rules):
    """dX's extension is H^T here, d_out / lambda2 wide: its steps lie in the last slices."""
    from paper_2407_17029_amd import binding as qb
    from gpu_util import f32_to_dev, bf16_to_dev, assert_close_bf16, assert_close_f32, OracleWeight
    T, d_out, d_in, lam = 300, 2112, 1088, 8
    print(f"case dense slices, single matrix T={T} {d_out}x{d_in}", flush=True)
    assert rules.dense_pays_t(T, d_in, d_out, d_out // lam) and rules.dense_call_plan(T, d_in, d_out, d_out // lam, 8).splits > 1
    L = synth.make_layer(5300, T, d_out, d_in, 8, lam, lam)
    qw = qb.qblora_quantize_blockwise(f32_to_dev(L.W), 64, qb.QUANT_ABSMAX_CODEBOOK, codebook, tiled=False)
    Wt = OracleWeight(oracle, L.W, codebook).assert_same(qw).dequantize(oracle, 2)
    Hb = synth.f32_to_bf16_bits(synth.normal_f32(5301, 0, (d_in // lam, d_out // lam)) * np.float32(0.02))
    dX, dH = qb.qablora_linear_bwd(qw, bf16_to_dev(Hb), lam, lam, 0.5, bf16_to_dev(L.X), bf16_to_dev(L.dY))
    torch.cuda.synchronize()
    rX, rH = oracle.qa_backward(Wt, L.X, L.dY, Hb, lam, lam, 0.5)
    assert_close_bf16(dX, rX, "dX")
    assert_close_f32(dH, rH, "dH")


@pytest.mark.parametrize("form", ["none", "two", "single"])
def test_fewer_tokens_on_the_workspace_of_many(oracle, codebook, form):
    """A training loop allocates for its largest batch; the backward of a smaller one takes more slices here, and more
    partial sums than the largest does."""
    from paper_2407_17029_amd import binding as qb
    from gpu_util import f32_to_dev, bf16_to_dev, assert_close_bf16, assert_close_f32, OracleWeight
    d_out, d_in, most = 1024, 512, 600
    print(f"case one workspace, {form}", flush=True)
    L = synth.make_layer(5900, 300, d_out, d_in, 16, 2, 2, b_std=0.05)
    qw = qb.qblora_quantize_blockwise(f32_to_dev(L.W), 64, qb.QUANT_ABSMAX_CODEBOOK, codebook)
    Wt = OracleWeight(oracle, L.W, codebook).assert_same(qw).dequantize(oracle, 2)
    ad = qb.Adapter(bf16_to_dev(L.A), bf16_to_dev(L.B), 2, 2, 0.5) if form == "two" else None
    Hb = synth.f32_to_bf16_bits(synth.normal_f32(5901, 0, (d_in // 8, d_out // 8)) * np.float32(0.02))
    q = qw.c_struct()
    need = (int(qb.lib().qablora_linear_bwd_workspace_bytes(qb.C.byref(q), 8, 8, most)) if form == "single"
            else qb.qblora_linear_bwd_workspace_bytes(qw, ad, most))
    ws = torch.empty(need, dtype=torch.uint8, device=qw.codes.device)
    for T in (300, 200, 100):
        X, dY = bf16_to_dev(L.X[:T]), bf16_to_dev(L.dY[:T])
        if form == "single":
            dX, dH = qb.qablora_linear_bwd(qw, bf16_to_dev(Hb), 8, 8, 0.5, X, dY, workspace=ws)
            torch.cuda.synchronize()
            rX, rH = oracle.qa_backward(Wt, L.X[:T], L.dY[:T], Hb, 8, 8, 0.5)
            assert_close_f32(dH, rH, "dH")
        else:
            dX, dA, dB = qb.qblora_linear_bwd(qw, ad, X, dY, need_grads=ad is not None, workspace=ws)
            torch.cuda.synchronize()
            A, B, s = (L.A, L.B, 0.5) if ad else (None, None, 0.0)
            rX, rA, rB = oracle.backward(Wt, L.X[:T], L.dY[:T], A, B, 2, 2, s)
            if ad:
                assert_close_f32(dA, rA, "dA")
                assert_close_f32(dB, rB, "dB")
        assert_close_bf16(dX, rX, f"dX, {T} tokens")


@pytest.mark.parametrize("form", ["two", "single"])
def test_gradients_alone_need_no_room_for_the_weight(codebook, form):
    """Without dX nothing is dequantized: the call takes a workspace smaller than the 16-bit weight, same bits."""
    from paper_2407_17029_amd import binding as qb
    from gpu_util import f32_to_dev, bf16_to_dev
    T, d_out, d_in = 200, 2048, 1024
    print(f"case gradients alone, {form}", flush=True)
    L = synth.make_layer(5950, T, d_out, d_in, 16, 2, 2, b_std=0.05)
    qw = qb.qblora_quantize_blockwise(f32_to_dev(L.W), 64, qb.QUANT_ABSMAX_CODEBOOK, codebook, qb.SCALES_E4M3_GROUPED)
    X, dY = bf16_to_dev(L.X), bf16_to_dev(L.dY)
    ws = torch.empty(2 * d_out * d_in - 256, dtype=torch.uint8, device=X.device)
    if form == "two":
        ad = qb.Adapter(bf16_to_dev(L.A), bf16_to_dev(L.B), 2, 2, 0.5)
        _, dA, dB = qb.qblora_linear_bwd(qw, ad, X, dY, need_dx=False, workspace=ws)
        _, rA, rB = qb.qblora_linear_bwd(qw, ad, X, dY)
        assert torch.equal(dA, rA) and torch.equal(dB, rB)
    else:
        H = torch.zeros((d_in // 8, d_out // 8), dtype=torch.bfloat16, device=X.device)
        _, dH = qb.qablora_linear_bwd(qw, H, 8, 8, 0.5, X, dY, need_dx=False, workspace=ws)
        _, rH = qb.qablora_linear_bwd(qw, H, 8, 8, 0.5, X, dY)
        assert torch.equal(dH, rH)


@pytest.mark.parametrize("fmt", ["nf4", "tile8"])
def test_codes_at_any_dword(codebook, fmt):
    """Codes that start between 16-byte boundaries: calls on fewer than 2048 tokens take them, in every form that reads
    codes, with the same results; calls on more refuse them."""
    from paper_2407_17029_amd import binding as qb
    from gpu_util import f32_to_dev
    d_out, d_in = 2112, 1088
    print(f"case codes placement {fmt}", flush=True)
    W = synth.base_weight(5990, 0, d_out, d_in)
    if fmt == "nf4":
        qw = qb.qblora_quantize_blockwise(f32_to_dev(W), 64, qb.QUANT_ABSMAX_CODEBOOK, codebook, tiled=False)
    else:
        qw = qb.qblora_quantize_blockwise(f32_to_dev(W), 64, qb.QUANT_MINMAX_INT4, block_rows=8, tiled=False)
    buf = torch.empty(qw.codes.numel() + 16, dtype=torch.uint8, device=qw.codes.device)
    moved = qb.QWeight(d_out, d_in, 64, qw.codebook, buf[4:4 + qw.codes.numel()].view_as(qw.codes), qw.scales, qw.beta,
                       block_rows=qw.block_rows)
    moved.codes.copy_(qw.codes)
    assert moved.codes.data_ptr() % 16 == 4
    g = torch.Generator(device="cuda").manual_seed(5991)
    X = torch.randn((2048, d_in), generator=g, device="cuda").to(torch.bfloat16)
    dY = torch.randn((2048, d_out), generator=g, device="cuda").to(torch.bfloat16)
    for T in (5, 100, 256, 300, 2047):
        assert torch.equal(qb.qblora_linear_fwd(moved, None, X[:T]), qb.qblora_linear_fwd(qw, None, X[:T]))
        dX = [qb.qblora_linear_bwd(w, None, X[:T], dY[:T], need_grads=False)[0] for w in (moved, qw)]
        assert torch.equal(*dX)
    Y = [qb.qblora_linear_fwd_noalloc(w, None, X, torch.empty((2048, d_out), dtype=torch.bfloat16, device="cuda")) for w in (moved, qw)]
    assert torch.equal(*Y)
    with pytest.raises(RuntimeError):
        qb.qblora_linear_fwd(moved, None, X)
    with pytest.raises(RuntimeError):
        qb.qblora_linear_bwd(moved, None, X, dY, need_grads=False)
