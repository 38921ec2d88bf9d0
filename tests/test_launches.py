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


FULL = {"workload": "gmm_full", "steps": [3]}


def _full(d, local, chains, **problem):
    return {**FULL, "args": {"d": d, "K": 5, "n_chains": chains, "n_steps": 3, "c_tilde": 1.0},
            "with": {"local": local, "n_leapfrog": 2 if local == "hmc" else 0}, "problem": problem}


def _step_kernel(run):
    assert run["init"] == 0 and run["step"] == [0]
    name, grid, block, lds = run["step_launches"][-1]
    return name, lds


def _is_split(name):
    return name.startswith("_ZN7restore11step_kernel") and name.split("EEEv")[0].endswith("ELb1")


def test_which_populations_read_the_slab_half_from_lds(tmp_path):
    # (d, move, Metropolis-Hastings) and the fewest chains that take the split
    limits = [(4, "rwmh", False, 81920), (5, "hmc", False, 81920), (6, "hmc", False, 131073), (7, "hmc", False, None),
              (8, "mala", False, 81920), (9, "rwmh", False, 131073), (10, "rwmh", False, 131073),
              (10, "mala", False, 81920), (11, "rwmh", False, 65536), (16, "hmc", False, 65536),
              (3, "mala", False, None), (4, "mala", True, 65537), (10, "rwmh", True, 65537), (11, "mala", True, 65536)]
    runs, want = [], []
    for d, local, mh, limit in limits:
        kw = {"c_tilde": 0.0, "large_step_prob": 0.3} if mh else {}
        for n in (limit - 1, limit) if limit else (65536, 1 << 20):
            runs.append(_full(d, local, n, **kw))
            want.append(bool(limit) and n >= limit)
    # (parameters staged in LDS: no split)
    runs.append(_full(8, "mala", 1 << 20, flags=1))
    want.append(False)
    for run, rec, split in zip(runs, record(tmp_path, runs), want):
        name, lds = _step_kernel(rec)
        assert _is_split(name) == split, (run, name)
        assert (lds > 0) == (split or run["problem"].get("flags") == 1), (run, lds)
