"""Step kernels that read a full-covariance slab half from the scalar cache
and half from LDS, for every move at the dimensions whose kernels are
compiled for different numbers of waves, with the learned regeneration
distribution behind the slab in LDS, and in batches that mix it with the
uniform one -- against ranges of the population small enough for the kernels
that read the scalar cache alone: every chain the same bits.  From d = 4 on
between two rows of the factor and all but the first come from LDS; below
there is no such kernel."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KEYS = ("x", "logp", "n_done", "t_done", "a_done", "status", "t_cur")
CHAINS = (1 << 17) + 65


@pytest.fixture(scope="module")
def R():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2409_07148_amd import restore
    return restore


def _arrays(R, prob, steps):
    run = R.Run(prob)
    run.step(steps)
    run.drain()
    arr = {k: v.cpu().numpy().copy() for k, v in run.arrays().items() if k in KEYS}
    run.close()
    return arr


def _workload(d, K, local, chains, c_factor):
    from workloads import gmm_full
    wl = gmm_full(d, K, chains, 12, problem_seed=240 + d, seed=250 + K, c_tilde=1.0)
    c, w = wl.params["covs"], wl.params["weights"]
    peak = float((w * (2 * np.pi) ** (-d / 2) / np.sqrt(np.linalg.det(c))).sum())
    return wl.with_(local=local, step=0.02 if local == "rwmh" else 0.005, n_leapfrog=2 if local == "hmc" else 0,
                    drain_cap=16, c_tilde=peak * c_factor)


def _mu(wl, K, seed):
    rng = np.random.default_rng(seed)
    at = np.arange(K) % wl.K
    sd = np.sqrt(np.array([np.diag(s) for s in wl.params["covs"]]))[at]
    return {"logits": rng.standard_normal(K), "means": wl.params["means"][at] + 0.5 * sd * rng.standard_normal((K, wl.d)),
            "log_std": np.log(sd), "beta": 0.2}


def _same_in_parts(R, wl, **kw):
    whole = _arrays(R, R.problem_from_workload(wl, **kw), 12)
    cuts = np.linspace(0, CHAINS, 4).astype(int)
    parts = [_arrays(R, R.problem_from_workload(wl, n_chains=int(hi - lo), first_chain=int(lo), **kw), 12)
             for lo, hi in zip(cuts[:-1], cuts[1:])]
    assert max(np.diff(cuts)) < 1 << 16
    for key in KEYS:
        assert np.array_equal(whole[key], np.concatenate([p[key] for p in parts], axis=-1)), key
    assert whole["n_done"].sum() > CHAINS


@pytest.mark.parametrize("d,K,local", [
    (4, 1, "mala"), (6, 5, "rwmh"), (6, 7, "hmc"), (8, 9, "hmc"), (10, 3, "rwmh"), (10, 64, "mala"), (10, 5, "hmc"),
    (11, 2, "mala"), (11, 7, "hmc"), (12, 5, "mala"), (12, 16, "hmc"), (13, 3, "hmc"), (14, 3, "rwmh"), (14, 5, "mala"),
    (14, 2, "hmc"), (15, 1, "rwmh"), (15, 5, "mala"), (15, 3, "hmc"), (16, 7, "mala"), (16, 64, "hmc")])
def test_restore_moves(R, d, K, local):
    _same_in_parts(R, _workload(d, K, local, CHAINS, 1e-2))


@pytest.mark.parametrize("d,K,local", [(6, 3, "mala"), (11, 5, "hmc"), (12, 2, "mala"), (14, 9, "hmc"), (16, 5, "hmc")])
def test_metropolis_hastings_moves(R, d, K, local):
    wl = _workload(d, K, local, CHAINS, 0.0)
    whole = _arrays(R, R.problem_from_workload(wl, large_step_prob=0.3), 12)
    cut = CHAINS // 3
    parts = [_arrays(R, R.problem_from_workload(wl, n_chains=hi - lo, first_chain=lo, large_step_prob=0.3), 12)
             for lo, hi in ((0, cut), (cut, 2 * cut), (2 * cut, CHAINS))]
    for key in KEYS:
        assert np.array_equal(whole[key], np.concatenate([p[key] for p in parts], axis=-1)), key


@pytest.mark.parametrize("K,mu_K,local", [(1, 64, "mala"), (7, 1, "mala"), (64, 64, "rwmh"), (16, 3, "rwmh")])
def test_learned_mu(R, K, mu_K, local):
    wl = _workload(8, K, local, CHAINS, 1.0)
    _same_in_parts(R, wl, mu=_mu(wl, mu_K, 17 * K + mu_K))


@pytest.mark.parametrize("block,buckets", [(128, 0), (256, 1)])
def test_batch_of_uniform_and_learned_mu(R, block, buckets):
    sizes = [(2, 5, 0), (8, 7, 64), (8, 3, 0), (2, 9, 3), (16, 5, 0), (8, 64, 1), (12, 6, 0)]
    wls = [_workload(d, K, "rwmh", 20011 + 64 * i, 1e-2) for i, (d, K, _) in enumerate(sizes)]
    mus = [_mu(wl, k, 30 + i) if k else None for i, (wl, (_, _, k)) in enumerate(zip(wls, sizes))]
    assert sum(w.n_chains for w in wls) > 1 << 17
    b = R.Batch(wls, n_steps=12, mus=mus)
    b.set_tiling(block, R.BATCH_ORDER_LPT, buckets)
    b.run()
    for i, (wl, mu) in enumerate(zip(wls, mus)):
        got = {k: v.cpu().numpy() for k, v in b.chain_sums(i).items()}
        ref = _arrays(R, R.problem_from_workload(wl, target_id=i, mu=mu), 12)
        for key in ("n_done", "t_done", "a_done", "t_cur"):
            assert np.array_equal(got[key], ref[key]), (wl.d, wl.K, key)
