"""Workloads whose speed matters to a user of the restore library.

Three kinds of work, each through the Python binding's public objects:

  * "run":   one whole run of a chain population (restore.Run: x_0 ~ mu,
             steps, drain, estimate, and the image estimate where the run has
             an image), a restore run or, with c_factor 0, the
             Metropolis-Hastings baseline with its burn-in.  The program has
             the problem's descriptors in hand; the run's buffers are its own.
  * "batch": one pass over many targets (restore.Batch, built once) and its
             estimates.
  * "train": one optimiser epoch of the learned regeneration distribution
             (learned_mu.MlpGmm: forward, loss and gradient on recorded
             samples, backward, Adam).

A run returns its estimate and the state of every chain; chains are exact
functions of (seed, chain, target), so whole numbers among them are too.
"""
import math

import numpy as np
import torch

from paper_2409_07148_amd import restore as R
from paper_2409_07148_amd.learned_mu import MlpGmm
from workloads import batched_uneven, gmm_full, gmm_iso_2d_unadjusted, pss_render

RUN = dict(kind="run", target="full", d=8, K=16, local="mala", step=0.005, leapfrog=0, chains=1 << 20, steps=512,
           burn=0, large=0.0, c_factor=1.0, mu_K=0, image_w=0, image_h=0, image_batches=0, tile=0)


def _run(**kw):
    return {**RUN, **kw}


def listed():
    return [
        # a quick look at a 2-D density: the smallest calls, where launches and host time count
        _run(name="small_2d", target="iso", d=2, K=4, local="rwmh", step=0.02, chains=2048, steps=200),
        # the 2-D workload: a few waves, one dependent step after another
        _run(name="iso_2d", target="iso", d=2, K=4, local="rwmh", step=0.02, chains=4096, steps=1000),
        # the general restore process on it (jumps without acceptance test)
        _run(name="unadjusted_2d", target="iso_unadjusted", d=2, K=4, local="rw_unadjusted", step=0.02, chains=4096,
             steps=1000),
        # a mid-sized population of odd sizes with Hamiltonian moves
        _run(name="hmc_5d", d=5, K=7, local="hmc", step=0.005, leapfrog=8, chains=30011, steps=300, c_factor=1e-3),
        # the 8-D workload at its provable c~: nearly every step a regeneration
        _run(name="mala_8d"),
        # the same at the c~ that serves its error best: long tours, local moves
        _run(name="mala_8d_long_tours", c_factor=1e-4),
        # the 8-D workload regenerating from a learned mixture of 64 components
        _run(name="learned_8d", mu_K=64),
        # the Metropolis-Hastings baseline: every step a gradient
        _run(name="baseline_8d", chains=1 << 18, steps=512, burn=1000, large=0.3, c_factor=0.0),
        # the 12-D rendering-shaped integrand into a 512 x 512 image, 16 batch images
        _run(name="image_12d", target="pss", d=12, K=0, local="rwmh", step=0.02, steps=256, image_w=512, image_h=512,
             image_batches=16),
        # the same stratified by 64-pixel tiles
        _run(name="image_tiles_12d", target="pss", d=12, K=0, local="rwmh", step=0.02, steps=256, image_w=512,
             image_h=512, image_batches=16, tile=64),
        # 256 uneven targets in one pass (their sizes and parameters fixed, the chains' seeds not)
        dict(name="batch_256", kind="batch", problem=1005, targets=256, chains_lo=1 << 10, chains_hi=1 << 18, steps=256, block=256,
             buckets=0),
        # a training epoch on four recorded steps of 2^20 chains
        dict(name="train_8d", kind="train", d=8, K=64, rows=1, samples=1 << 22, hidden=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["small", "full", "full", "learned", "baseline", "image", "batch", "train"])
    if kind == "small":
        if rng.random() < 0.3:
            return _run(target="iso_unadjusted", d=2, K=4, local="rw_unadjusted", step=0.02,
                        chains=_log_int(rng, 256, 8192), steps=rng.randint(50, 1000))
        return _run(target="iso", d=rng.randint(1, 4), K=rng.randint(1, 8), local=rng.choice(["rwmh", "mala"]),
                    step=rng.choice([0.01, 0.02]), chains=_log_int(rng, 256, 60000), steps=rng.randint(50, 1000))
    if kind == "full":
        local = rng.choice(["rwmh", "mala", "hmc"])
        return _run(d=rng.randint(2, 16), K=rng.randint(2, 32), local=local, step=0.02 if local == "rwmh" else 0.005,
                    leapfrog=rng.randint(2, 8) if local == "hmc" else 0, chains=_log_int(rng, 1 << 12, 1 << 18),
                    steps=rng.randint(50, 300), c_factor=rng.choice([1.0, 1e-2, 1e-4]))
    if kind == "learned":
        return _run(d=rng.choice([2, 8]), K=rng.randint(2, 32), local=rng.choice(["rwmh", "mala"]), step=0.005,
                    chains=_log_int(rng, 1 << 14, 1 << 20), steps=rng.randint(50, 512), mu_K=rng.randint(3, 64),
                    c_factor=rng.choice([1.0, 1e-4]))
    if kind == "baseline":
        return _run(d=rng.randint(2, 12), K=rng.randint(2, 24), local=rng.choice(["rwmh", "mala"]), step=0.005,
                    chains=_log_int(rng, 1 << 12, 1 << 17), steps=rng.randint(50, 512), burn=rng.randint(100, 1000),
                    large=0.3, c_factor=0.0)
    if kind == "image":
        w, h = rng.randint(64, 512), rng.randint(64, 512)
        return _run(target="pss", d=12, K=0, local="rwmh", step=0.02, chains=_log_int(rng, 1 << 15, 1 << 20),
                    steps=rng.randint(20, 256), image_w=w, image_h=h, image_batches=rng.randint(1, 16),
                    tile=rng.choice([0, 0, 32, 64]))
    if kind == "batch":
        return dict(kind="batch", problem=rng.randint(1, 1 << 20), targets=_log_int(rng, 8, 200), chains_lo=1 << 8,
                    chains_hi=_log_int(rng, 1 << 12, 1 << 17), steps=rng.randint(50, 256),
                    block=rng.choice([64, 128, 256]), buckets=rng.choice([0, 1]))
    return dict(kind="train", d=rng.randint(2, 16), K=rng.randint(3, 64), rows=_log_int(rng, 1, 32),
                samples=_log_int(rng, 1 << 12, 1 << 18), hidden=rng.choice([33, 64, 64, 128]))


# --- inputs -----------------------------------------------------------------

def _peak_full(p, d):
    """An upper bound of the mixture: the sum of its components' peaks."""
    return float((p["weights"] * (2 * math.pi) ** (-d / 2) / np.sqrt(np.linalg.det(p["covs"]))).sum())


def _workload(c, seed):
    """The run's workload: parameters and chain seed from `seed`, c_tilde by
    the lifetime rule (mean lifetime at most an eighth of the budget under an
    upper bound of the density), scaled by c_factor."""
    d, K, B = c["d"], c["K"], c["steps"]
    kw = dict(local=c["local"], step=c["step"], n_leapfrog=c["leapfrog"])
    if c["target"] == "full":
        wl = gmm_full(d, K, c["chains"], B, problem_seed=1002 + seed, seed=2002 + seed, c_tilde=1.0)
        bound = _peak_full(wl.params, d)
    elif c["target"] == "pss":
        wl = pss_render(c["chains"], B, problem_seed=1003 + seed, seed=2003 + seed, image=(c["image_w"], c["image_h"]),
                        image_batches=c["image_batches"])
        p = wl.params
        bound = ((1 + np.abs(p["tex_a_amp"]).sum() / 8) * (1 + np.abs(p["tex_b_amp"]).sum() / 8)
                 * (float(p["base"][0]) + 2 * float((p["lobe_weights"] * p["lobe_kappa"]).sum())))
        kw["tile_px"] = c["tile"]
    elif c["target"] == "iso_unadjusted":
        # its c_tilde belongs to its one parameter set; the chains differ by seed
        return gmm_iso_2d_unadjusted(c["chains"], B, seed=2001 + seed)
    else:
        rng = np.random.default_rng(1001 + seed)
        w = rng.dirichlet(np.full(K, 4.0))
        params = {"weights": w, "means": rng.uniform(0.2, 0.8, size=(K, d)), "sigmas": np.full(K, 0.05)}
        wl = gmm_full(1, 1, c["chains"], B, seed=2001 + seed).with_(target="gmm_iso", d=d, K=K, params=params)
        bound = float((w * (2 * math.pi * 0.05 ** 2) ** (-d / 2)).sum())
    ct = max(1.0, 8.0 * bound / B) * c["c_factor"]
    return wl.with_(c_tilde=float(f"{ct:.3g}"), **kw)


def _learned_mu(wl, K, seed):
    """A mixture as training leaves it: diagonal components at the target's
    modes, their scales near the modes' marginal ones, a defensive share."""
    rng = np.random.default_rng(3004 + seed)
    sd = np.sqrt(np.array([np.diag(s) for s in wl.params["covs"]]))
    at = np.arange(K) % wl.K
    logits = np.log(wl.params["weights"][at] + 1e-6) + 0.3 * rng.standard_normal(K)
    means = wl.params["means"][at] + 0.5 * sd[at] * rng.standard_normal((K, wl.d))
    log_std = np.log(sd[at]) + 0.1 * rng.standard_normal((K, wl.d))
    return {"logits": logits, "means": means, "log_std": log_std, "beta": 0.1}


def prepare(case, seed):
    c = case
    if c["kind"] == "run":
        wl = _workload(c, seed % 100003)
        kw = {}
        if c["mu_K"]:
            kw["mu"] = _learned_mu(wl, c["mu_K"], seed % 100003)
            kw["c_tilde"] = wl.c_tilde / 0.1
        if c["large"]:
            kw["large_step_prob"] = c["large"]
        return {"case": c, "problem": R.problem_from_workload(wl, **kw)}
    if c["kind"] == "batch":
        wls = batched_uneven(c["targets"], problem_seed=c["problem"], seed=2005 + seed % 100003, n_steps=c["steps"],
                             chains_lo=c["chains_lo"], chains_hi=c["chains_hi"])
        b = R.Batch(wls, n_steps=c["steps"])
        b.set_tiling(c["block"], R.BATCH_ORDER_LPT, c["buckets"])
        return {"case": c, "batch": b}
    return {"case": c, **_training(c, seed)}


def _training(c, seed):
    """A model in the middle of its training and the samples it is fitted
    to: states of chains near the modes with Exp(1) holding times."""
    d, K, G, n = c["d"], c["K"], c["rows"], c["samples"]
    model = MlpGmm(d=d, K=K, hidden=c["hidden"], G=G, seed=3004 + seed % 100003)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda")  # noqa: E731
    randn = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    modes, sd = 0.2 + 0.6 * rand(16, d), torch.exp(math.log(0.01) + math.log(10.0) * rand(16, d))
    at = torch.arange(K, device="cuda") % 16
    b3 = model.theta[-model.O:]
    b3[:K] = 0.5 * randn(K)
    b3[K:K + K * d] = (modes[at] + 0.5 * sd[at] * randn(K, d)).reshape(-1)
    b3[K + K * d:] = (torch.log(sd[at]) + 0.2 * randn(K, d)).reshape(-1)
    model.m.copy_(1e-3 * randn(model.n_params))
    model.v.copy_(1e-6 * (0.5 + rand(model.n_params)))
    model.t = 100
    xs, ws = [], []
    for _ in range(G):
        pick = torch.randint(16, (n,), generator=g, device="cuda")
        xs.append((modes[pick] + sd[pick] * randn(n, d)).clamp_(2.0 ** -24, 1.0))
        ws.append(-torch.log(rand(n).clamp_(min=2.0 ** -24)))
    return {"model": model, "xs": xs, "ws": ws}


# --- one pass ---------------------------------------------------------------

def run(state):
    c = state["case"]
    if c["kind"] == "run":
        r = R.Run(state["problem"])
        if c["burn"]:
            r.step(c["burn"])
            r.reset_sums()
        r.step(c["steps"])
        r.drain()
        out = {"estimate": _numbers(r.estimate())}
        a = r.arrays()
        for k in ("x", "logp", "a_done", "t_done", "n_done", "status"):
            out[k] = a[k]
        if r.image is not None:
            out["image"] = r.image
            out["mean"], out["se"] = r.image_estimate()
        r.close()
        return out
    if c["kind"] == "batch":
        b = state["batch"]
        b.run()
        est = [_numbers(e) for e in b.estimates()]
        sums = [b.chain_sums(i) for i in range(b.n)]
        return {"estimates": {k: np.stack([e[k] for e in est]) for k in ("values", "counts")},
                "n_done": torch.cat([s["n_done"] for s in sums]), "t_done": torch.cat([s["t_done"] for s in sums]),
                "a_done": torch.cat([s["a_done"] for s in sums])}
    m = state["model"]
    m.forward()
    for g in range(m.G):
        m.nll_and_grad(state["xs"][g], state["ws"][g], g)
    m.backward()
    m.adam(1e-3)
    return {"out": m.out, "loss": m.loss, "dout": m.dout, "grad": m.grad, "theta": m.theta, "m": m.m, "v": m.v}


def _numbers(est):
    """An estimate's floating values and its whole numbers, as arrays."""
    return {"values": np.array([v for v in est.values() if isinstance(v, float)], dtype=np.float64),
            "counts": np.array([v for v in est.values() if isinstance(v, int)], dtype=np.int64)}


# --- what a pass cannot do without -------------------------------------------

def _step_flops(c, d, K, grad):
    """One transition: the density at the new state (an FMA counts two, a
    transcendental one), its gradient where every move needs it, the learned
    mixture's density, the clocks and the move."""
    if c.get("target") == "pss":
        return 8 * 7 + 8 * 15 + 3 * 21 + 30 + 4 * d
    if c.get("target") == "full":
        f = K * (d * d + 3 * d + 7 + (d * d + 2 * d if grad else 0))
    else:
        f = K * (3 * d + 7 + (3 * d if grad else 0))
        if c.get("target") == "iso_unadjusted":
            f += K * (13 * d + 8)
    return f + c.get("mu_K", 0) * (3 * d + 7) + 30 + 4 * d


def work(case):
    c = case
    if c["kind"] == "run":
        d, n = c["d"], c["chains"]
        moves = c["c_factor"] == 0.0
        f = _step_flops(c, d, c["K"], moves and c["local"] != "rwmh") * n * (c["steps"] + c["burn"])
        pixels = c["image_w"] * c["image_h"]
        return {"bytes": n * (4 * d + 36) + 4 * pixels * (max(1, c["image_batches"]) + 2), "flops": f}
    if c["kind"] == "batch":
        # uniform d in 2..16 and K in 2..32, chains uniform in their logarithm
        mean = (c["chains_hi"] - c["chains_lo"]) / math.log(c["chains_hi"] / c["chains_lo"])
        per = np.mean([_step_flops({"target": "full"}, d, K, False) for d in range(2, 17) for K in range(2, 33)])
        return {"bytes": c["targets"] * mean * 28, "flops": c["targets"] * mean * c["steps"] * per}
    d, K, n = c["d"], c["K"], c["samples"] * c["rows"]
    H, O = c["hidden"], K * (1 + 2 * d)
    params = 12 * H + H * H + O * H + 2 * H + O
    # scores, squares and log-sum-exp; responsibility-weighted moments; the MLP both ways
    return {"bytes": 4 * n * (d + 1) + 28 * params, "flops": n * K * (4 * d + 6 + 4 * d) + 6 * params * c["rows"]}


# --- the same in 64 bits, where that has a value -------------------------------

def exact(case, seed):
    """A training epoch in float64.  (A chain is a long sequence of
    decisions: its sums have no value but the ones its own random numbers
    give.)"""
    if case["kind"] != "train":
        return None
    s = _training(case, seed)
    m = s["model"]
    d, K, H, O = m.d, m.K, m.hidden, m.O
    theta = m.theta.double().requires_grad_()
    ctx, at, parts = m.ctx.double(), 0, []
    for rows, cols in ((H, m.in_dim), (H, H), (O, H)):
        parts += [theta[at:at + rows * cols].view(rows, cols), theta[at + rows * cols:at + rows * cols + rows]]
        at += rows * cols + rows
    gelu = torch.nn.functional.gelu
    out = gelu(gelu(ctx @ parts[0].t() + parts[1]) @ parts[2].t() + parts[3]) @ parts[4].t() + parts[5]
    leaf = out.detach().requires_grad_()
    beta = float(np.float32(m.beta))
    loss = torch.zeros(m.G, dtype=torch.float64, device="cuda")
    chunk = 1 << 17
    for g in range(m.G):
        W = s["ws"][g].double().sum()
        for i in range(0, s["ws"][g].numel(), chunk):
            x, w = s["xs"][g][i:i + chunk].double(), s["ws"][g][i:i + chunk].double()
            row = leaf[g]
            lpi = torch.log_softmax(row[:K], 0) + math.log1p(-beta)
            mean, ls = row[K:K + K * d].view(K, d), row[K + K * d:].view(K, d)
            q = torch.zeros(x.shape[0], K, dtype=torch.float64, device="cuda")
            for j in range(d):
                q = q + ((x[:, j:j + 1] - mean[None, :, j]) * torch.exp(-ls[None, :, j])) ** 2
            a = lpi - 0.5 * d * math.log(2 * math.pi) - ls.sum(1) - 0.5 * q
            a = torch.cat([a, torch.full((x.shape[0], 1), math.log(beta), dtype=torch.float64, device="cuda")], 1)
            part = -(w * torch.logsumexp(a, 1)).sum() / W
            part.backward()
            loss[g] += part.detach()
    out.backward(leaf.grad)
    grad = theta.grad
    b1, b2, eps, t = 0.9, 0.999, 1e-8, m.t + 1
    m1 = b1 * m.m.double() + (1 - b1) * grad
    v1 = b2 * m.v.double() + (1 - b2) * grad * grad
    new = theta.detach() - 1e-3 * (m1 / (1 - b1 ** t)) / (torch.sqrt(v1 / (1 - b2 ** t)) + eps)
    return {"out": out.detach(), "loss": loss, "dout": leaf.grad, "grad": grad, "theta": new, "m": m1, "v": v1}
