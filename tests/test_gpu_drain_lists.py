"""Drains of large populations, whose lists go from one lane a chain to four
once they are short, against drains of parts of them with one lane a chain
throughout: every chain the same bits.  The cases differ in how many chains
are left when: few from the start, a list that becomes short between
launches, one that stays long to the end, one that lasts through several
launches of four lanes a chain."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KEYS = ("x", "logp", "logu", "n_done", "t_done", "a_done", "status", "t_cur", "a_cur", "last_dt")
SHORT = 16384   # the longest list that takes four lanes a chain


@pytest.fixture(scope="module")
def R():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2409_07148_amd import restore
    return restore


def _workload(d, K, local, chains, share, cap):
    """Broad components, and a c_tilde at which `share` of the box has a
    killing rate below 1: that share survives a step more often than not."""
    from workloads import gmm_full
    wl = gmm_full(d, K, chains, 4, problem_seed=180 + d, seed=190 + K, c_tilde=1.0)
    params = dict(wl.params, covs=wl.params["covs"] * 20.0)
    x = np.random.default_rng(d).random((4000, d))
    logp = np.full(4000, -np.inf)
    for w, m, c in zip(params["weights"], params["means"], params["covs"]):
        v = np.linalg.solve(np.linalg.cholesky(c), (x - m).T)
        logp = np.logaddexp(logp, np.log(w) - 0.5 * d * np.log(2 * np.pi) - 0.5 * np.linalg.slogdet(c)[1]
                            - 0.5 * (v ** 2).sum(0))
    return wl.with_(params=params, local=local, step=0.02 if local == "rwmh" else 0.005, drain_cap=cap,
                    n_leapfrog=2 if local == "hmc" else 0, c_tilde=float(np.exp(np.quantile(logp, 1.0 - share))))


def _run(R, prob):
    run = R.Run(prob)
    run.step(4)
    run.drain()
    est = run.estimate()
    arr = {k: v.cpu().numpy().copy() for k, v in run.arrays().items() if k in KEYS}
    run.close()
    return arr, {k: est[k] for k in ("transitions", "accepts", "kills", "tours_done", "tours_censored")}


@pytest.mark.parametrize("d,K,local,chains,share,cap,left", [
    (1, 3, "rwmh", 65536, 0.015, 40, "crossing"), (5, 9, "mala", 70001, 0.05, 300, "short"),
    (8, 16, "mala", 140000, 0.3, 300, "crossing"), (13, 5, "hmc", 66000, 0.05, 100, "short"),
    (16, 7, "rwmh", 90001, 0.055, 200, "crossing"), (12, 64, "mala", 66000, 0.03, 64, "short"),
    (3, 4, "hmc", 131072, 0.9, 40, "long"), (2, 5, "rwmh", 65599, 0.02, 1100, "short")])
def test_drain_gives_the_same_chains(R, d, K, local, chains, share, cap, left):
    wl = _workload(d, K, local, chains, share, cap)
    whole, est = _run(R, R.problem_from_workload(wl))
    # chains still in their tours after the first launches of 1, 2, 4, ... steps
    alive = [_run(R, R.problem_from_workload(wl, drain_cap=n))[1]["tours_censored"] for n in (1, 3, 7, 15, 31, 63, 127)
             if n <= cap]
    if left == "short":
        assert 1000 < alive[0] <= SHORT
    elif left == "crossing":
        assert alive[0] > SHORT and any(100 < n <= SHORT for n in alive[1:])
    else:
        assert alive[-1] > SHORT
    cuts = np.linspace(0, chains, 2 + chains // 60000).astype(int)
    parts = [_run(R, R.problem_from_workload(wl, n_chains=int(hi - lo), first_chain=int(lo), flags=R.FLAG_INLINE_RNG))
             for lo, hi in zip(cuts[:-1], cuts[1:])]
    for key in KEYS:
        assert np.array_equal(whole[key], np.concatenate([p[0][key] for p in parts], axis=-1)), key
    for key in est:
        assert est[key] == sum(p[1][key] for p in parts), key
