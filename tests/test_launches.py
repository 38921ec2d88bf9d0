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


def test_which_small_populations_take_four_lanes(tmp_path):
    # (d, move, K) and the most chains that do
    limits = [(2, "rwmh", 1, 0), (2, "rwmh", 2, 8192), (3, "rwmh", 16, 12288), (4, "rwmh", 3, 16384),
              (2, "mala", 5, 16384), (2, "mala", 7, 32768), (5, "hmc", 2, 8192), (5, "hmc", 3, 16384),
              (5, "hmc", 7, 32768), (8, "hmc", 5, 12288), (8, "hmc", 7, 16384), (12, "rwmh", 3, 16384),
              (12, "mala", 5, 12288), (13, "rwmh", 7, 16384),
              (6, "mala", 7, 16384), (6, "mala", 16, 32768)]
    runs, want = [], []
    for d, local, K, limit in limits:
        for n in (limit, limit + 1) if limit else (500,):
            run = _full(d, local, n)
            run["args"]["K"] = K
            run["with"]["drain_cap"] = 40
            runs.append({**run, "drain": True})
            want.append(n <= limit)
    for run, rec, lanes in zip(runs, record(tmp_path, runs), want):
        for launch, kernel in ((rec["step_launches"][-1], "step_pre_kernel"), (rec["drain_launches"][-1], "drain_pre_kernel")):
            name, grid, block, lds = launch
            n, d = run["args"]["n_chains"], run["args"]["d"]
            assert kernel in name and (lds > 0) == lanes and f"ELi{4 if lanes else 1}EEEv" in name, (run, launch)
            # a workgroup of 256 once the lanes fill half the SIMDs
            threads = n * (4 if lanes else 1)
            assert block == (256 if threads > 32768 else 64), (run, launch)
            if kernel == "drain_pre_kernel":
                assert grid == -(-threads // block)
