"""Kernels that spread a chain over several lanes -- the steps and the drain
of small populations (four lanes for full-covariance mixtures, sixteen for
the unadjusted jump process) and the short lists of a large population's
drain -- against the kernels of one lane a chain: the same arithmetic in the
same order, so the same bits.  Component counts below, at and past a pass
of four (and of four or eight for the jump process), every log-sum-exp block
size, the smallest and largest dimension, ragged last waves."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KEYS = ("x", "logp", "logu", "n_done", "t_done", "a_done", "status", "t_cur", "a_cur", "last_dt")


@pytest.fixture(scope="module")
def R():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2409_07148_amd import restore
    return restore


def _run(R, prob, steps):
    run = R.Run(prob)
    for n in steps:
        run.step(n)
    run.drain()
    est = run.estimate()
    arr = {k: v.cpu().numpy().copy() for k, v in run.arrays().items() if k in KEYS}
    run.close()
    return arr, {k: est[k] for k in ("transitions", "accepts", "kills", "tours_done", "tours_censored")}


def _same(a, b):
    for key in KEYS:
        assert np.array_equal(a[0][key], b[0][key], equal_nan=True), key
    assert a[1] == b[1]


def _full(d, K, local, chains, n_steps, drain_cap):
    from workloads import gmm_full
    wl = gmm_full(d, K, chains, n_steps, problem_seed=80 + d, seed=90 + K, c_tilde=1.0)
    c, w = wl.params["covs"], wl.params["weights"]
    peak = float((w * (2 * np.pi) ** (-d / 2) / np.sqrt(np.linalg.det(c))).sum())
    return wl.with_(local=local, step=0.02 if local == "rwmh" else 0.005, n_leapfrog=3 if local == "hmc" else 0,
                    drain_cap=drain_cap, c_tilde=1e-3 * peak)


@pytest.mark.parametrize("d,K,local", [
    (1, 1, "rwmh"), (1, 5, "mala"), (2, 2, "rwmh"), (3, 3, "mala"), (4, 4, "rwmh"), (5, 7, "hmc"), (6, 6, "rwmh"),
    (8, 16, "mala"), (8, 5, "hmc"), (9, 9, "mala"), (12, 64, "rwmh"), (16, 2, "mala"), (16, 64, "hmc")])
def test_small_population_full(R, d, K, local):
    # FLAG_INLINE_RNG keeps the kernels of one lane a chain
    wl = _full(d, K, local, 1003, 20, 40)
    _same(_run(R, R.problem_from_workload(wl), (13, 7)),
          _run(R, R.problem_from_workload(wl, flags=R.FLAG_INLINE_RNG), (20,)))


@pytest.mark.parametrize("d,K", [(1, 1), (1, 8), (1, 9), (2, 1), (2, 4), (2, 5), (2, 9)])
def test_small_population_unadjusted(R, d, K):
    from workloads import gmm_iso_2d_unadjusted
    rng = np.random.default_rng(7 * K + d)
    params = {"weights": rng.dirichlet(np.full(K, 4.0)), "means": rng.uniform(0.2, 0.8, size=(K, d)),
              "sigmas": np.full(K, 0.08)}
    wl = gmm_iso_2d_unadjusted(517, 30).with_(d=d, K=K, params=params, drain_cap=30, c_tilde=40.0)
    _same(_run(R, R.problem_from_workload(wl), (11, 19)),
          _run(R, R.problem_from_workload(wl, flags=R.FLAG_INLINE_RNG), (30,)))


@pytest.mark.parametrize("d,K,local,chains", [(2, 3, "rwmh", 70001), (5, 9, "mala", 70001), (8, 16, "mala", 140000),
                                              (13, 5, "hmc", 66000)])
def test_drain_of_a_large_population(R, d, K, local, chains):
    # ranges of the population too small for the large population's drain
    wl = _full(d, K, local, chains, 4, 60)
    whole, est = _run(R, R.problem_from_workload(wl), (4,))
    cuts = np.linspace(0, chains, 2 + chains // 60000).astype(int)
    parts = [_run(R, R.problem_from_workload(wl, n_chains=int(hi - lo), first_chain=int(lo), flags=R.FLAG_INLINE_RNG),
                  (4,)) for lo, hi in zip(cuts[:-1], cuts[1:])]
    for key in KEYS:
        assert np.array_equal(whole[key], np.concatenate([p[0][key] for p in parts], axis=-1)), key
    for key in est:
        assert est[key] == sum(p[1][key] for p in parts), key


@pytest.mark.parametrize("d,K,local", [(1, 1, "rwmh"), (2, 2, "mala"), (2, 3, "rwmh"), (2, 4, "rwmh"), (3, 5, "mala"),
                                       (4, 3, "hmc"), (6, 9, "rwmh"), (16, 6, "mala")])
def test_small_population_isotropic(R, d, K, local):
    # the first four components held in registers, a chunk's steps in pairs
    # of buffers and the odd ones after them
    from workloads import gmm_iso_2d
    rng = np.random.default_rng(11 * K + d)
    params = {"weights": rng.dirichlet(np.full(K, 4.0)), "means": rng.uniform(0.2, 0.8, size=(K, d)),
              "sigmas": np.full(K, 0.1)}
    wl = gmm_iso_2d(1003, 23).with_(d=d, K=K, params=params, local=local, step=0.02, drain_cap=40, c_tilde=0.05,
                                    n_leapfrog=2 if local == "hmc" else 0)
    ref = _run(R, R.problem_from_workload(wl, flags=R.FLAG_INLINE_RNG), (23,))
    _same(_run(R, R.problem_from_workload(wl), (1, 15, 7)), ref)
