"""Densities at the ends of float32's range with four lanes a chain against
one lane: a component so narrow that its exponent overflows everywhere (one
component, a filler beside it in its log-sum-exp block), some of several
such, and weights of zero."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KEYS = ("x", "logp", "logu", "n_done", "t_done", "a_done", "status", "t_cur", "a_cur", "last_dt")


@pytest.mark.parametrize("d,local", [(2, "rwmh"), (2, "mala"), (3, "hmc"), (9, "mala"), (13, "rwmh")])
@pytest.mark.parametrize("sigmas", [(1e-21,), (1e-21, 0.1), (0.1, 0.1, 1e-21), (1e-21,) * 3, (0.1, 0.1, 0.1, 0.1, 1e-21)])
def test_overflowing_components(d, local, sigmas):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2409_07148_amd import restore as R
    from workloads import gmm_full
    K = len(sigmas)
    rng = np.random.default_rng(100 * K + d)
    w = np.full(K, 1.0 / K)
    w[-1] = 0.0 if K == 3 else w[-1]
    params = {"weights": w, "means": rng.uniform(0.2, 0.8, size=(K, d)),
              "covs": np.stack([np.eye(d) * s * s for s in sigmas])}
    wl = gmm_full(d, K, 515, 12, seed=6, c_tilde=1.0).with_(params=params, local=local, drain_cap=20, c_tilde=0.3,
                                                             n_leapfrog=2 if local == "hmc" else 0)
    got = []
    for flags in (0, R.FLAG_INLINE_RNG):
        run = R.Run(R.problem_from_workload(wl, flags=flags))
        run.step(12)
        run.drain()
        est = run.estimate()
        got.append(({k: v.cpu().numpy().copy() for k, v in run.arrays().items() if k in KEYS},
                    [est[k] for k in ("transitions", "accepts", "kills", "tours_done", "tours_censored", "nonfinite")]))
        run.close()
    for k in KEYS:
        assert np.array_equal(got[0][0][k], got[1][0][k], equal_nan=True), k
    assert got[0][1] == got[1][1]
