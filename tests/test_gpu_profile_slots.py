"""Which event slots a call records, and that the launch which a slot names lies between its events."""
import pytest
import torch

from paper_2407_17029_amd import synth

pytestmark = pytest.mark.gpu


def recorded(qb, call, slots):
    """The slots among `slots` whose events `call` recorded."""
    def events():
        pair = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        for e in pair:
            e.record()                                        # creates the native handles
        return pair
    pairs, mark = {s: events() for s in slots}, torch.cuda.Event(enable_timing=True)
    call()                                                    # (first use of a kernel: its attributes are set)
    torch.cuda.synchronize()
    mark.record()
    for s, p in pairs.items():
        qb.qblora_profile_events(s, *p)
    try:
        call()
    finally:
        for s in slots:
            qb.qblora_profile_events(s, None, None)
    torch.cuda.synchronize()
    return {s for s, p in pairs.items() if mark.elapsed_time(p[0]) > 0 and p[0].elapsed_time(p[1]) > 0}


@pytest.mark.parametrize("lam1", [1, 4, 8, 16])
@pytest.mark.parametrize("T", [64, 520])
def test_dequantize_slot_of_a_single_matrix_forward(codebook, rules, T, lam1):
    """At 520 tokens the weight is dequantized once, in the launch of the pooling (lambda1 up to 8) or behind the re-layouts."""
    from gpu_util import bf16_to_dev, f32_to_dev
    qb, (d_out, d_in) = rules.qb, (512, 1024)
    L = synth.make_layer(2100, T, d_out, d_in, 8, 1, 1)
    qw = qb.qblora_quantize_blockwise(f32_to_dev(L.W), 64, qb.QUANT_ABSMAX_CODEBOOK, codebook)
    X, H = bf16_to_dev(L.X), torch.zeros((d_in // lam1, d_out // 2), dtype=torch.bfloat16, device="cuda")
    once = rules.dense_pays(T, d_out, d_in, d_in // lam1) and T > 256
    assert once == (T == 520)
    assert recorded(qb, lambda: qb.qablora_linear_fwd(qw, H, lam1, 2, 0.5, X), [qb.PROFILE_DEQUANT]) == ({qb.PROFILE_DEQUANT} if once else set())
