"""The host side of a run on the CPU: which kernels it launches for which
population, and what a failing launch returns (HIP calls recorded, no device
work)."""
import pytest

from tests.launches import record

E_HIP = -3


@pytest.mark.parametrize("kw", [
    {"workload": "gmm_iso_2d", "args": {"n_chains": 300, "n_steps": 10}},
    # fixed-point sums: a launch more
    {"workload": "pss_render", "args": {"n_chains": 3000, "n_steps": 8, "image": [32, 32]}, "problem": {"flags": 32}}])
def test_init_returns_the_error_of_each_of_its_launches(tmp_path, kw):
    whole, = record(tmp_path, [kw])
    n = len(whole["init_launches"])
    assert whole["init"] == 0 and n >= 2
    failing = record(tmp_path, [{**kw, "fail_at": i} for i in range(n)])
    assert [r["init"] for r in failing] == [E_HIP] * n
