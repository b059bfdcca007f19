"""Which event slots a call records, and that the launch which a slot names lies between its events."""
import pytest
import torch

from paper_2407_17029_amd import synth

pytestmark = pytest.mark.gpu


def timed_pair():
    pair = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for e in pair:
        e.record()                                            # creates the native handles
    return pair


def recorded(qb, call, slots, pairs=None):
    """The slots among `slots` whose events `call` recorded."""
    pairs, mark = pairs or [timed_pair() for _ in slots], torch.cuda.Event(enable_timing=True)
    call()                                                    # (first use of a kernel: its attributes are set)
    torch.cuda.synchronize()
    mark.record()
    for s, p in zip(slots, pairs):
        qb.qblora_profile_events(s, *p)
    try:
        call()
    finally:
        for s in slots:
            qb.qblora_profile_events(s, None, None)
    torch.cuda.synchronize()
    return {s for s, p in zip(slots, pairs) if mark.elapsed_time(p[0]) > 0 and p[0].elapsed_time(p[1]) > 0}


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


@pytest.mark.parametrize("T,d_out,d_in,R,lam,once,together", [
    (64, 512, 512, 16, 1, False, True), (70, 512, 2752, 40, 2, False, True),       # not sliced; in slices
    (64, 512, 512, 16, 4, False, False),                                           # A is copied: the narrow GEMM waits
    (520, 512, 512, 16, 2, True, False),                                           # not sliced: no sums for the weight to go with
    (520, 1024, 4096, 64, 2, True, True), (520, 1024, 4096, 64, 4, True, False),
])
def test_slots_of_a_forward(codebook, rules, T, d_out, d_in, R, lam, once, together):
    """The re-layouts and the weight's pass, alone or in launches of the narrow GEMM: their pairs lie where their launches do."""
    from gpu_util import adapter_to_dev, bf16_to_dev, f32_to_dev
    qb = rules.qb
    L = synth.make_layer(2110, T, d_out, d_in, R, lam, lam)
    qw = qb.qblora_quantize_blockwise(f32_to_dev(L.W), 64, qb.QUANT_ABSMAX_CODEBOOK, codebook)
    ad, X = adapter_to_dev(L, lam, lam, 0.5), bf16_to_dev(L.X)
    assert once == (T > 256 and rules.dense_pays(T, d_out, d_in, R))
    slots = [qb.PROFILE_ADAPTER_FWD, qb.PROFILE_PREP, qb.PROFILE_DEQUANT]
    narrow, prep, weight = pairs = [timed_pair() for _ in slots]
    assert recorded(qb, lambda: qb.qblora_linear_fwd(qw, ad, X), slots, pairs) == {*slots[:2], *(slots[2:] if once else [])}
    inside = lambda a, b: b[0].elapsed_time(a[0]) >= 0 and a[1].elapsed_time(b[1]) >= 0
    assert inside(prep, narrow) == together
    if not together:
        assert prep[1].elapsed_time(narrow[0]) >= 0
    if once:
        assert inside(weight, narrow) == together and inside(weight, prep) == (not together)
