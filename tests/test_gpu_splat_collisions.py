"""The accumulation of binned image splats where many records fall on a few
pixels of a band that is large enough for compare-and-swap, against the same
run's sums in fixed point: waves whose lanes collide leave off swapping, and
no record may be lost on the way."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size,batches,sigma", [(128, 1, 0.0005), (128, 1, 0.003), (96, 3, 0.02), (64, 1, 1e-5)])
def test_image_on_a_few_pixels(size, batches, sigma):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2409_07148_amd import restore as R
    from workloads import pss_render
    chains, steps = 3000, 20
    wl = pss_render(chains, steps, problem_seed=17, seed=18, image=(size, size), image_batches=batches)
    wl = wl.with_(step=1e-4)   # local moves stay within their pixel
    ls = np.full((4, 12), np.log(0.3))
    ls[:, :2] = np.log(sigma)
    mu = {"logits": np.zeros(4), "means": np.random.default_rng(1).uniform(0.3, 0.7, (4, 12)), "log_std": ls, "beta": 0.1}
    # holding times of about 0.01 at the regenerated states: far above the
    # fixed point's unit of 2^-32
    kw = {"mu": mu, "c_tilde": 100.0 * sigma ** 2}
    imgs = []
    for flags in (0, R.FLAG_IMAGE_FIXED):
        run = R.Run(R.problem_from_workload(wl, flags=flags, **kw))
        run.step(steps)
        imgs.append(run.image.cpu().numpy().astype(np.float64))
        run.close()
    got, ref = imgs
    # most of what the chains spend their time on lies on few pixels
    top = np.sort(ref.ravel())[::-1]
    assert top[:size * size // 8].sum() > 0.5 * top.sum() > 0
    # n additions in float32, each rounded by at most 2^-24 of the running sum,
    # independently: six standard deviations; n roundings to 2^-33 in fixed point
    n = chains * (steps + 1)
    assert np.all(np.abs(got - ref) <= 6.0 * np.sqrt(n) * 2.0 ** -24 * ref + n * 2.0 ** -33)
