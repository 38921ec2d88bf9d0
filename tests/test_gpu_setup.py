"""The parameters a run starts with, which a small slab takes through the
setup kernel's arguments (up to 960 floats) and a larger one through a copy:
log p of the initial states against float64, for slabs of one component, at
either side of the limit and of the largest size."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# 156 floats a component at d = 16 (6: 936, 7: 1092), 48 at d = 8 (20: 960, 21: 1008)
@pytest.mark.parametrize("d,K", [(1, 1), (8, 20), (8, 21), (16, 6), (16, 7), (16, 64)])
def test_initial_log_density(d, K):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2409_07148_amd import restore as R
    from workloads import gmm_full
    run = R.Run(R.problem_from_workload(gmm_full(d, K, 777, 4, problem_seed=3 + d, seed=5, c_tilde=1.0)))
    arr = {k: v.cpu().numpy().astype(np.float64) for k, v in run.arrays().items()}
    p = gmm_full(d, K, 777, 4, problem_seed=3 + d, seed=5, c_tilde=1.0).params
    x, u = arr["x"].T, 2.0 ** -24
    a, err = np.empty((777, K)), np.empty((777, K))
    for k in range(K):
        L = np.linalg.cholesky(p["covs"][k])
        W = np.linalg.inv(L)
        dx = x - p["means"][k]
        v = dx @ W.T
        a[:, k] = np.log(p["weights"][k]) - 0.5 * d * np.log(2 * np.pi) - np.log(np.diag(L)).sum() - 0.5 * (v ** 2).sum(1)
        # W, mean and difference rounded once each, d products summed; then d squares summed
        ev = (d + 4) * u * ((np.abs(dx) + u) @ np.abs(W.T))
        err[:, k] = (np.abs(v) * ev + 0.5 * ev ** 2).sum(1) + 0.5 * (d + 4) * u * (v ** 2).sum(1) + 4 * u * np.abs(a[:, k])
    m = a.max(1, keepdims=True)
    w = np.exp(a - m)
    ref = m[:, 0] + np.log(w.sum(1))
    # the log-sum-exp passes its terms' errors on with their weights (twice, for
    # their change) and adds a few roundings of its own
    tol = 2 * (w * err).sum(1) / w.sum(1) + (K + 8) * u + 4 * u * np.abs(ref)
    assert np.all(np.abs(arr["logp"] - ref) <= tol), float(np.max(np.abs(arr["logp"] - ref) / tol))
    run.close()
