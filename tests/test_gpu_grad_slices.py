"""Parameter gradients in a single slice of the tokens, which are written without a reduction, beside ones in several; and the
reduction with and without the weight's dequantize pass in its launch: the same bits."""
import pytest
import torch

from paper_2407_17029_amd import binding as qb
from test_gpu_layer import _setup
from test_gpu_qablora import _setup as _setup_qa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d_out,d_in,R,lam1,lam2", [
    (130, 320, 448, 24, 2, 4), (64, 192, 576, 8, 16, 8), (200, 704, 192, 136, 8, 16), (33, 256, 512, 16, 32, 2),
    (97, 512, 320, 40, 4, 32), (1, 64, 64, 8, 1, 1), (1000, 16512, 64, 256, 2, 2),
])
def test_adapter(oracle, codebook, T, d_out, d_in, R, lam1, lam2):
    from gpu_util import assert_close_bf16, assert_close_f32
    print(f"case slices T={T} {d_out}x{d_in} R={R} lam=({lam1},{lam2})", flush=True)
    L, qw, Wt, ad, X, dY = _setup(qb, oracle, codebook, 9000 + T, T, d_out, d_in, R, lam1, lam2, 0.5)
    dX, dA, dB = qb.qblora_linear_bwd(qw, ad, X, dY)
    _, dA2, dB2 = qb.qblora_linear_bwd(qw, ad, X, dY, need_dx=False)     # without the weight in the reduction's launch
    torch.cuda.synchronize()
    rX, rA, rB = oracle.backward(Wt, L.X, L.dY, L.A, L.B, lam1, lam2, 0.5)
    assert_close_bf16(dX, rX, "dX")
    assert_close_f32(dA, rA, "dA")
    assert_close_f32(dB, rB, "dB")
    assert torch.equal(dA, dA2) and torch.equal(dB, dB2)


@pytest.mark.parametrize("T,d_out,d_in,lam", [(64, 320, 192, 2), (10, 64, 64, 8), (190, 4224, 2176, 1)])
def test_single_matrix_adapter_in_one_slice(oracle, codebook, T, d_out, d_in, lam):
    from gpu_util import assert_close_bf16, assert_close_f32
    print(f"case slices qa T={T} {d_out}x{d_in} lam={lam}", flush=True)
    L, qw, Wt, Hb, H, X, dY = _setup_qa(qb, oracle, codebook, 9100 + T, T, d_out, d_in, lam, lam, minmax=True)
    buf = torch.full((H.numel() + 9,), 7.0, dtype=torch.float32, device=X.device)
    rX, rH = oracle.qa_backward(Wt, L.X, L.dY, Hb, lam, lam, 0.5)
    first = None
    for off in (0, 1):                                   # on a 16-byte boundary: written without a reduction
        dX, dH = qb.qablora_linear_bwd(qw, H, lam, lam, 0.5, X, dY, dH=buf[off:off + H.numel()].view(H.shape))
        torch.cuda.synchronize()
        assert_close_bf16(dX, rX, "dX")
        assert_close_f32(dH, rH, "dH")
        assert torch.all(buf[off + H.numel():] == 7.0)
        first = dH.clone() if first is None else first
        assert torch.equal(dH, first)
        buf.fill_(7.0)
