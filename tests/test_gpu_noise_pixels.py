"""Noise of images that the histogram route does not hold, by selection over
their pixels: that they are, is read back; lists of few keys, lists that
overflow a workgroup's staging, ties down to the last digit, medians between
two far values, images of one piece to 256 and more pieces than workgroups.
sigma, set size and step count equal the oracle's exactly."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _image(kind, n, seed):
    rng = np.random.default_rng(seed)
    z = rng.standard_normal(n)
    if kind == "two_scales":  # half of the pixels a million times narrower than the others
        return np.where(rng.random(n) < 0.5, 1e-6 * z, z)
    if kind == "bimodal":  # two equal groups: the median falls between them
        return np.where(np.arange(n) % 2 == 0, -50.0, 50.0) + 0.01 * z
    if kind == "normal":
        return z
    if kind == "exponential":
        return rng.exponential(1.0, n)
    if kind == "clump":  # 14 000 values within the first 22 bits of one key, the median among them
        x = np.where(np.arange(n) % 2 == 0, -1.0, 1.0) * rng.uniform(2.0, 3e4, n)
        x[rng.choice(n, 14000, replace=False)] = 1.0 + 1e-4 * rng.random(14000)
        return x
    raise ValueError(kind)


# (a narrow clip of many steps visits more places than the histogram route keeps)
@pytest.mark.parametrize("kind,dtype,kappa,steps,n_img,n", [
    ("two_scales", "float32", 3.0, 10, 1, 40001), ("two_scales", "float32", 1.5, 100, 100, 140001),
    ("bimodal", "float32", 3.0, 10, 1, 500001), ("bimodal", "float16", 3.0, 10, 1, 4194304),
    ("clump", "float32", 0.9, 100, 1, 50001), ("normal", "float16", 1.5, 100, 3, 1000003),
    ("exponential", "float32", 1.5, 100, 1, 1000003)])
def test_images_solved_from_their_pixels(kind, dtype, kappa, steps, n_img, n):
    import torch
    import paper_2503_08854_amd as dt
    host = [_image(kind, n, 10 * k + n).astype(dtype) for k in range(min(n_img, 4))]
    want = [oracle.mad_noise(x.astype(np.float32), kappa, steps) for x in host]
    dev = [torch.from_numpy(x).cuda().view(1, n) for x in host]
    ctx = dt.Context(0)
    assert dt.debug_noise_pixels(ctx) == 0
    sig, used, it = dt.image_noise(ctx, [dev[k % len(dev)] for k in range(n_img)], kappa, steps)
    assert dt.debug_noise_pixels(ctx) == n_img
    got = list(zip(sig.cpu().tolist(), used.cpu().tolist(), it.cpu().tolist()))
    assert got == [want[k % len(want)] for k in range(n_img)]
    plain = torch.randn((1, n), device="cuda")
    dt.image_noise(ctx, [plain])
    assert dt.debug_noise_pixels(ctx) == 0
    ctx.close()
