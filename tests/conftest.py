import ctypes as C
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def oracle():
    import oracle as o
    o.lib()
    return o


@pytest.fixture(scope="session")
def codebook():
    from paper_2407_17029_amd import synth
    return synth.codebook_nf4_style()


class DensePlan(C.Structure):
    _fields_ = [("shape", C.c_int), ("splits", C.c_int), ("ns", C.c_int64)]


@pytest.fixture(scope="session")
def rules():
    """The library's own rules, by their C++ names."""
    from paper_2407_17029_amd import binding as qb
    L = qb.lib()
    pays = L["_ZN6qblora10dense_paysEliii"]
    pays.argtypes, pays.restype = [C.c_int64, C.c_int, C.c_int, C.c_int], C.c_bool
    pays_t = L["_ZN6qblora12dense_pays_tEliii"]
    pays_t.argtypes, pays_t.restype = [C.c_int64, C.c_int, C.c_int, C.c_int], C.c_bool
    plan = L["_ZN6qblora10dense_planEliiii"]
    plan.argtypes, plan.restype = [C.c_int64, C.c_int, C.c_int, C.c_int, C.c_int], DensePlan
    call_plan = L["_ZN6qblora15dense_call_planEliiii"]
    call_plan.argtypes, call_plan.restype = plan.argtypes, DensePlan
    few = L["_ZN6qblora11few_appliesElii"]
    few.argtypes, few.restype = [C.c_int64, C.c_int, C.c_int], C.c_bool
    return type("Rules", (), dict(qb=qb, L=L, dense_pays=pays, dense_pays_t=pays_t, dense_plan=plan, dense_call_plan=call_plan,
                                   few_applies=few))
