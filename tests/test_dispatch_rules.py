"""The host-side rules that choose a kernel form or size its scratch.  They depend on sizes only: no GPU is needed."""
import ctypes as C

import pytest


class DensePlan(C.Structure):
    _fields_ = [("shape", C.c_int), ("splits", C.c_int), ("ns", C.c_int64)]


@pytest.fixture(scope="module")
def rules():
    """The library's own rules, by their C++ names."""
    from paper_2407_17029_amd import binding as qb
    L = qb.lib()
    pays = L["_ZN6qblora10dense_paysEliii"]
    pays.argtypes, pays.restype = [C.c_int64, C.c_int, C.c_int, C.c_int], C.c_bool
    plan = L["_ZN6qblora10dense_planEliiii"]
    plan.argtypes, plan.restype = [C.c_int64, C.c_int, C.c_int, C.c_int, C.c_int], DensePlan
    return type("Rules", (), dict(qb=qb, L=L, dense_pays=pays, dense_plan=plan))


@pytest.mark.parametrize("T,d_out,d_in,K2,dense", [
    (300, 22016, 8192, 0, False), (512, 22016, 8192, 128, False), (700, 16384, 8192, 128, False),
    (512, 16384, 8192, 1024, False),
    (512, 4096, 4096, 0, True), (1337, 5120, 5120, 64, True), (2048, 22016, 8192, 0, True), (8192, 4096, 4096, 128, True),
])
def test_forward_dequantizes_first_only_where_it_pays(rules, T, d_out, d_in, K2, dense):
    """22016 x 8192 at 512 tokens: 190 us from the codes, 265 us dequantized first."""
    assert rules.dense_pays(T, d_out, d_in, K2) == dense


SHAPES = [(64, 64), (512, 512), (1000, 768), (4096, 4096), (11008, 4096), (4096, 11008), (5120, 13824), (13824, 5120),
          (19200, 768), (22016, 8192), (8192, 22016)]


def _weight(qb, d_out, d_in, grouped=False, block_rows=1, block=64):
    q = qb.CQWeight()
    q.d_out, q.d_in, q.block, q.block_rows = d_out, d_in, block, block_rows
    q.codes = q.scales = 0x1000                          # never dereferenced
    if grouped:
        q.scale_mode, q.scale_group = qb.SCALES_E4M3_GROUPED, 256
        q.scale_codes = q.scale_step = q.scale_mid = 0x1000
    return q


@pytest.mark.parametrize("d_out,d_in", SHAPES)
@pytest.mark.parametrize("kind", ["plain", "grouped", "8x4"])
def test_inference_workspace_serves_smaller_batches(rules, d_out, d_in, kind):
    q = _weight(rules.qb, d_out, d_in, kind == "grouped", *((8, 32) if kind == "8x4" else ()))
    need = [rules.L.qblora_linear_decode_tokens_workspace_bytes(C.byref(q), T) for T in range(0, 300)]
    assert all(a <= b for a, b in zip(need, need[1:]))
    assert need[256] == need[299]
