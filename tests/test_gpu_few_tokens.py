"""GPU parity: the forward for at most 256 tokens whose waves split the contraction, at the edges of its tiles."""
import pytest
import torch

from paper_2407_17029_amd import synth

pytestmark = pytest.mark.gpu

# T, d_out, d_in, R, format: 32 x 32, 32 x 64 and 64 x 64 tiles; fewer steps than waves, one, and a ragged last round
CASES = [
    (1, 64, 64, 0, "nf4"),
    (33, 128, 576, 8, "nf4"),           # ragged tokens, nine steps, extension in the tenth
    (256, 576, 448, 136, "grouped"),    # seven steps, three extension steps, the last one partial
    (31, 8256, 1088, 72, "minmax"),     # 32 x 64
    (130, 4160, 704, 24, "tile8"),      # 64 x 64, ragged tokens
    (130, 4160, 640, 0, "tile8_nf4"),
]


@pytest.mark.parametrize("T,d_out,d_in,R,fmt", CASES)
def test_waves_split_the_contraction(oracle, codebook, rules, T, d_out, d_in, R, fmt):
    from paper_2407_17029_amd import binding as qb
    from gpu_util import f32_to_dev, bf16_to_dev, assert_close_bf16, OracleWeight
    print(f"case few T={T} {d_out}x{d_in} R={R} {fmt}", flush=True)
    assert rules.few_applies(T, d_out, d_in)
    L = synth.make_layer(7100 + T + d_out, T, d_out, d_in, max(R, 8), 2, 2)
    br = 8 if fmt.startswith("tile8") else 1
    minmax, grouped = fmt in ("minmax", "tile8"), fmt == "grouped"
    if minmax:
        qw = qb.qblora_quantize_blockwise(f32_to_dev(L.W), 64, qb.QUANT_MINMAX_INT4, block_rows=br)
    else:
        qw = qb.qblora_quantize_blockwise(f32_to_dev(L.W), 64, qb.QUANT_ABSMAX_CODEBOOK, codebook,
                                          qb.SCALES_E4M3_GROUPED if grouped else qb.SCALES_FP32, block_rows=br)
    torch.cuda.synchronize()
    Wt = OracleWeight(oracle, L.W, codebook, minmax, grouped, br).assert_same(qw).dequantize(oracle, 2)
    ad = qb.Adapter(bf16_to_dev(L.A), bf16_to_dev(L.B), 2, 2, 0.5) if R else None
    A, B, s = (L.A, L.B, 0.5) if R else (None, None, 0.0)
    X = bf16_to_dev(L.X)
    Y = torch.full((T, d_out), float("nan"), dtype=torch.bfloat16, device=X.device)
    qb.qblora_linear_fwd(qw, ad, X, Y=Y)
    Y2 = torch.empty_like(Y)
    qb.qblora_linear_fwd_noalloc(qw, ad, X, Y2)
    torch.cuda.synchronize()
    assert_close_bf16(Y, oracle.forward(Wt, L.X, A, B, 2, 2, s), "Y")
    assert torch.equal(Y.view(torch.int16), Y2.view(torch.int16))


def test_single_matrix_adapter_on_grouped_scales(oracle, codebook, rules):
    """The single-matrix forward reconstructs the grouped block scales for this kernel; the extension is H's."""
    from paper_2407_17029_amd import binding as qb
    from gpu_util import f32_to_dev, bf16_to_dev, assert_close_bf16, OracleWeight
    T, d_out, d_in, lam = 130, 576, 832, 8
    print(f"case few, single matrix on grouped scales T={T} {d_out}x{d_in}", flush=True)
    assert rules.few_applies(T, d_out, d_in)
    L = synth.make_layer(7200, T, d_out, d_in, 8, lam, lam)
    qw = qb.qblora_quantize_blockwise(f32_to_dev(L.W), 64, qb.QUANT_ABSMAX_CODEBOOK, codebook, qb.SCALES_E4M3_GROUPED)
    torch.cuda.synchronize()
    Wt = OracleWeight(oracle, L.W, codebook, False, True).assert_same(qw).dequantize(oracle, 2)
    Hb = synth.f32_to_bf16_bits(synth.normal_f32(7201, 0, (d_in // lam, d_out // lam)) * 0.02)
    Y = qb.qablora_linear_fwd(qw, bf16_to_dev(Hb), lam, lam, 0.5, bf16_to_dev(L.X))
    torch.cuda.synchronize()
    assert_close_bf16(Y, oracle.qa_forward(Wt, L.X, Hb, lam, lam, 0.5), "Y")


@pytest.mark.parametrize("T,d_out,d_in", [(21, 37, 1024), (150, 37, 2048), (250, 130, 1088)])
def test_mid_batch_slices_of_odd_outputs(oracle, codebook, T, d_out, d_in):
    """Inference above 16 tokens on layers whose outputs are no whole words: the slices' sum takes its scalar path."""
    from paper_2407_17029_amd import binding as qb
    from gpu_util import f32_to_dev, bf16_to_dev, assert_close_bf16, OracleWeight
    print(f"case mid batch, odd outputs T={T} {d_out}x{d_in}", flush=True)
    L = synth.make_layer(7300 + T, T, d_out, d_in, 8, 1, 1)
    qw = qb.qblora_quantize_blockwise(f32_to_dev(L.W), 64, qb.QUANT_ABSMAX_CODEBOOK, codebook)
    Y = torch.full((T, d_out), float("nan"), dtype=torch.bfloat16, device=qw.codes.device)
    qb.qblora_linear_decode(qw, bf16_to_dev(L.X), Y=Y)
    torch.cuda.synchronize()
    Wt = OracleWeight(oracle, L.W, codebook).assert_same(qw).dequantize(oracle, 2)
    assert_close_bf16(Y, oracle.forward(Wt, L.X, None, None, 1, 1, 0.0), "Y")


def test_mid_batch_on_the_workspace_of_the_largest(oracle, codebook):
    """A serving loop allocates for 256 tokens once; this layer needs no partial tiles there, and three slices at 100."""
    from paper_2407_17029_amd import binding as qb
    from gpu_util import f32_to_dev, bf16_to_dev, assert_close_bf16, OracleWeight
    d_out, d_in = 19200, 768
    print(f"case mid batch, one workspace {d_out}x{d_in}", flush=True)
    L = synth.make_layer(7500, 100, d_out, d_in, 8, 1, 1)
    qw = qb.qblora_quantize_blockwise(f32_to_dev(L.W), 64, qb.QUANT_ABSMAX_CODEBOOK, codebook)
    q = qw.c_struct()
    need = int(qb.lib().qblora_linear_decode_tokens_workspace_bytes(qb.C.byref(q), 256))
    ws = torch.empty(max(need, 256), dtype=torch.uint8, device=qw.codes.device)
    Wt = OracleWeight(oracle, L.W, codebook).assert_same(qw).dequantize(oracle, 2)
    for T in (100, 33, 17):                              # (up to 16 tokens the weight is not rounded, and there are no slices)
        Y = qb.qblora_linear_decode(qw, bf16_to_dev(L.X[:T]), workspace=ws)
        torch.cuda.synchronize()
        assert_close_bf16(Y, oracle.forward(Wt, L.X[:T], None, None, 1, 1, 0.0), f"Y, {T} tokens")


def test_mid_batch_of_four_gibibytes(codebook):
    """256 rows of 2^23 inputs: more than the kernel's 32-bit row offsets reach, so the call goes in two halves."""
    from paper_2407_17029_amd import binding as qb
    T, d_out, d_in = 256, 8, 1 << 23
    print(f"case mid batch of 4 GiB T={T} {d_out}x{d_in}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(7600)
    W = torch.randn((d_out, d_in), generator=g, device="cuda").mul_(0.02)
    qw = qb.qblora_quantize_blockwise(W, 64, qb.QUANT_ABSMAX_CODEBOOK, codebook, tiled=False)
    X = torch.empty((T, d_in), dtype=torch.bfloat16, device="cuda")
    for row in X:
        row.copy_(torch.randn((d_in,), generator=g, device="cuda"))
    Y = qb.qblora_linear_decode(qw, X)
    halves = [qb.qblora_linear_decode(qw, X[t:t + 128]) for t in (0, 128)]
    assert torch.equal(Y, torch.cat(halves))


@pytest.mark.parametrize("T,d_out,d_in", [(8, 40, 4160), (5, 4096, 8128), (8, 256, 6080)])
def test_sixteen_wave_decode_of_a_packed_model(oracle, codebook, T, d_out, d_in):
    """Packed INT4 model, few long rows: block counts (65, 127, 95) that the waves of a workgroup do not divide."""
    from paper_2407_17029_amd import binding as qb
    from gpu_util import f32_to_dev, bf16_to_dev, assert_close_bf16, OracleWeight
    print(f"case sixteen waves T={T} {d_out}x{d_in}", flush=True)
    L = synth.make_layer(7400 + d_in, T, d_out, d_in, 8, 1, 1)
    qw = qb.qblora_quantize_blockwise(f32_to_dev(L.W), 64, qb.QUANT_MINMAX_INT4)
    Y = torch.full((T, d_out), float("nan"), dtype=torch.bfloat16, device=qw.codes.device)
    qb.qblora_linear_decode(qw, bf16_to_dev(L.X), Y=Y, pack=qb.qblora_decode_pack(qw))
    torch.cuda.synchronize()
    Wt = OracleWeight(oracle, L.W, codebook, True).assert_same(qw).dequantize(oracle, 2)
    assert_close_bf16(Y, oracle.forward(Wt, L.X, None, None, 1, 1, 0.0), "Y")
