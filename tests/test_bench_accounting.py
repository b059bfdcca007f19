"""A launch that two event slots bracket counts once in the bench's per-projection times.  No GPU is needed."""
import pytest

MS = {"adapter_fwd": 1.0, "adapter_bwd": 2.0, "adapter_grads": 4.0, "prep": 8.0, "dequant_fwd": 8.0, "grad_reduce": 16.0,
      "dequant_bwd": 16.0}


@pytest.mark.parametrize("fwd,bwd,adapter,total", [(True, True, 7.0, 31.0), (True, False, 23.0, 31.0), (False, True, 15.0, 31.0),
                                                  (False, False, 31.0, 31.0)])
def test_shared_launches_count_once(fwd, bwd, adapter, total):
    import bench
    a, p = bench.side_launches(MS, {"dequant_fwd": fwd, "dequant_bwd": bwd})
    assert sum(a.values()) == adapter and sum(a.values()) + sum(p.values()) == total


@pytest.mark.parametrize("fwd,in_narrow,adapter,total", [
    (True, ["prep", "dequant_fwd"], {"adapter_fwd": 92.0, "prep": None}, 92 + 2 + 4 + 16 + 8),   # re-layouts and pass inside the 100 ms
    (False, ["prep"], {"adapter_fwd": 100.0, "prep": None}, 100 + 2 + 4 + 16),
    (False, [], {"adapter_fwd": 100.0, "prep": 8.0}, 100 + 2 + 4 + 8 + 16),
])
def test_launches_of_the_narrow_gemm_count_once(fwd, in_narrow, adapter, total):
    import bench
    a, p = bench.side_launches({**MS, "adapter_fwd": 100.0}, {"dequant_fwd": fwd, "dequant_bwd": False}, in_narrow)
    assert {k: a.get(k) for k in adapter} == adapter and sum(a.values()) + sum(p.values()) == total
