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
