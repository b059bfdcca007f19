"""Grouped E4M3 scales where a wave's group can go wrong: one scale, a group less or more than whole by one, a last
group that does not fill a workgroup, and groups whose scales are all equal.  Bit for bit against the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_out,d_in,flat", [(1, 64, False), (5, 3264, False), (1, 16448, False), (2, 33024, False),
                                             (1, 69504, False), (3, 8192, True)])
def test_scale_groups(oracle, codebook, d_out, d_in, flat):
    from paper_2407_17029_amd import binding as qb
    from gpu_util import f32_to_dev, OracleWeight
    print(f"case scale groups {d_out}x{d_in} flat={flat}", flush=True)
    rng = np.random.default_rng(8100 + d_in)
    W = (rng.standard_normal((d_out, d_in)) * 0.02).astype(np.float32)
    if flat:
        W = np.where(W > 0, np.float32(0.5), np.float32(-0.5))
    qw = qb.qblora_quantize_blockwise(f32_to_dev(W), 64, qb.QUANT_ABSMAX_CODEBOOK, codebook, qb.SCALES_E4M3_GROUPED)
    torch.cuda.synchronize()
    OracleWeight(oracle, W, codebook, False, True).assert_same(qw)
