"""Step kernels that read a full-covariance slab half from the scalar cache
and half from LDS (populations and batches of 2^16 chains and more) against
those that read it from the scalar cache alone (smaller ones): the same
arithmetic, so every chain's sums are the same bits.  Dimensions at the
edges of the LDS part (one, some and all rows of the factor; blocks padded
to 16 bytes or not), component counts around the log-sum-exp blocks, and a
last wave that is nearly empty."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KEYS = ("x", "logp", "n_done", "t_done", "a_done", "status", "t_cur")
CHAINS = (1 << 16) + 65


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


@pytest.mark.parametrize("d,K,local,c_factor", [
    (1, 1, "rwmh", 1.0), (2, 3, "mala", 1e-2), (3, 64, "rwmh", 1e-2), (4, 5, "hmc", 1e-2), (5, 9, "mala", 0.0),
    (7, 2, "mala", 1e-2), (8, 16, "mala", 1e-2), (8, 7, "mala", 0.0), (9, 3, "hmc", 1e-2), (12, 5, "rwmh", 0.0),
    (13, 2, "mala", 1e-2), (16, 64, "rwmh", 1e-2), (16, 3, "mala", 0.0)])
def test_split_slab_gives_the_same_chains(R, d, K, local, c_factor):
    from workloads import gmm_full
    wl = gmm_full(d, K, CHAINS, 24, problem_seed=40 + d, seed=50 + K, c_tilde=1.0)
    wl = wl.with_(local=local, step=0.02 if local == "rwmh" else 0.005, n_leapfrog=3 if local == "hmc" else 0,
                  drain_cap=32, c_tilde=_c_tilde(wl) * c_factor)
    kw = {"large_step_prob": 0.3} if c_factor == 0.0 else {}
    whole = _arrays(R, R.problem_from_workload(wl, **kw), wl.n_steps)
    cut = CHAINS // 2
    parts = [_arrays(R, R.problem_from_workload(wl, n_chains=hi - lo, first_chain=lo, **kw), wl.n_steps)
             for lo, hi in ((0, cut), (cut, CHAINS))]
    for key in KEYS:
        got = np.concatenate([p[key] for p in parts], axis=-1)
        assert np.array_equal(whole[key], got), key


def _c_tilde(wl):
    """About the largest density: its mixture's peaks, summed."""
    c, w = wl.params["covs"], wl.params["weights"]
    return float((w * (2 * np.pi) ** (-wl.d / 2) / np.sqrt(np.linalg.det(c))).sum())


@pytest.mark.parametrize("block,buckets", [(64, 1), (256, 0)])
def test_split_slab_in_a_batch(R, block, buckets):
    from workloads import gmm_full
    wls = []
    for i, (d, K) in enumerate([(1, 4), (2, 1), (4, 3), (5, 64), (8, 5), (9, 2), (12, 7), (13, 3), (16, 64)]):
        wl = gmm_full(d, K, 8191 + 31 * i, 20, problem_seed=60 + i, seed=70, c_tilde=1.0)
        wls.append(wl.with_(local="rwmh", step=0.02, drain_cap=16, c_tilde=_c_tilde(wl) * 1e-2))
    assert sum(w.n_chains for w in wls) >= 1 << 16
    b = R.Batch(wls, n_steps=20)
    b.set_tiling(block, R.BATCH_ORDER_LPT, buckets)
    b.run()
    for i, wl in enumerate(wls):
        got = {k: v.cpu().numpy() for k, v in b.chain_sums(i).items()}
        ref = _arrays(R, R.problem_from_workload(wl, target_id=i, integrand_p=True), 20)
        for key in ("n_done", "t_done", "a_done", "t_cur"):
            assert np.array_equal(got[key], ref[key]), (wl.d, key)
