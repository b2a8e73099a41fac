"""Iterated-MAD noise at the sizes and value distributions where the
histogram route can go wrong: images listed whole and just above that size,
unaligned buffers, ties too many to list, medians between far values, cuts
outside the histogram's range, and images its plan misses (solved from the
pixels).  sigma, set size and step count equal the oracle's exactly."""
import math

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _images(kind, n, rng):
    z = rng.standard_normal(n)
    if kind == "normal":
        return 3.0 + 0.7 * z
    if kind == "outliers":  # a fifth of the pixels far off: the clip moves over several steps
        return np.where(rng.random(n) < 0.2, 6.0 * np.abs(z) + 2.0, z)
    if kind == "integers":
        return np.rint(6.0 * z)
    if kind == "few_values":
        return rng.integers(0, 3, n).astype(float)
    if kind == "mostly_zero":
        return np.where(rng.random(n) < 0.6, 0.0, z)
    if kind == "constant":
        return np.full(n, -2.5)
    if kind == "two_scales":  # half of the pixels a million times narrower than the others
        return np.where(rng.random(n) < 0.5, 1e-6 * z, z)
    if kind == "bimodal":  # two equal groups: the median falls between them
        return np.where(np.arange(n) % 2 == 0, -50.0, 50.0) + 0.01 * z
    if kind == "masked":
        return np.where(rng.random(n) < 0.9, np.nan, z)
    if kind == "infinities":
        return np.where(rng.random(n) < 0.01, np.inf * np.sign(z), z)
    if kind == "huge":
        return np.where(rng.random(n) < 0.3, 3e38 * np.sign(z), 1e37 * z)
    if kind == "tiny":
        return 1e-41 * np.rint(100 * z)  # denormal FP32 values
    raise ValueError(kind)


KINDS = ["normal", "outliers", "integers", "few_values", "mostly_zero", "constant", "two_scales", "bimodal", "masked",
         "infinities", "huge", "tiny"]


@pytest.mark.parametrize("dtype", ["float32", "float16"])
@pytest.mark.parametrize("n", [1, 2, 3, 16383, 16384, 16385, 70001, 1000003])
def test_noise_routes_match_oracle(n, dtype):
    import torch
    import paper_2503_08854_amd as dt
    rng = np.random.default_rng(n)
    ctx = dt.Context(0)
    for kappa, steps in [(3.0, 10), (0.8, 10), (1e6, 4)]:
        host, dev = [], []
        for k, kind in enumerate(KINDS):
            with np.errstate(over="ignore"):
                x = _images(kind, n, rng).astype(dtype)
            # every image at another offset from 16-byte alignment
            buf = torch.zeros(n + 16, dtype=getattr(torch, dtype), device="cuda")
            view = buf[k % 8:k % 8 + n].view(1, n)
            view.copy_(torch.from_numpy(x).view(1, n))
            host.append(x)
            dev.append(view)
        sig, used, it = dt.image_noise(ctx, dev, kappa, steps)
        torch.cuda.synchronize()
        sig, used, it = sig.cpu().numpy(), used.cpu().numpy(), it.cpu().numpy()
        for k, x in enumerate(host):
            ws, wu, wi = oracle.mad_noise(x.astype(np.float32), kappa, steps)
            assert (used[k], it[k]) == (wu, wi), (KINDS[k], kappa, used[k], wu, it[k], wi)
            assert sig[k] == ws or (math.isnan(ws) and math.isnan(sig[k])), (KINDS[k], kappa, sig[k], ws)
    ctx.close()


@pytest.mark.parametrize("n_img,n,every", [(1, 4194304, 1), (1, 262145, 1), (5, 1000003, 5), (300, 16385, 7), (30, 70001, 1)])
def test_images_the_plan_misses_shared_by_workgroups(n_img, n, every):
    """Every `every`-th image is solved from its pixels: one by all workgroups,
    some among many, more pieces than workgroups; the calls follow one another
    with no synchronisation."""
    import torch
    import paper_2503_08854_amd as dt
    rng = np.random.default_rng(n_img + n)
    host = [_images("two_scales" if k % (2 * every) == 0 else "bimodal" if k % every == 0 else "normal", n,
                    rng).astype("float32") for k in range(n_img)]
    dev = [torch.from_numpy(x).cuda().view(1, n) for x in host]
    ctx = dt.Context(0)
    got = [dt.image_noise(ctx, dev, 3.0, 10) for _ in range(3)]
    torch.cuda.synchronize()
    want = [oracle.mad_noise(x, 3.0, 10) for x in host]
    for sig, used, it in got:
        assert sig.cpu().tolist() == [w[0] for w in want]
        assert used.cpu().tolist() == [w[1] for w in want]
        assert it.cpu().tolist() == [w[2] for w in want]
    ctx.close()
