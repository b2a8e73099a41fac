"""Noise of an image of more than 2^32 pixels, where 32-bit counts and ranks
wrap: sigma, set size and step count equal the FP64 definition's, evaluated
here on the number of pixels of each FP16 value (first checked against the
oracle on a small image)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _mad_of_counts(values, counts, kappa, steps):
    """Iterated MAD of an image given as sorted values and their numbers."""
    def middle(v, c):
        order = np.argsort(v, kind="stable")
        v, cum = v[order], np.cumsum(c[order])
        n = int(cum[-1])
        lo, hi = (v[np.searchsorted(cum, r, side="right")] for r in ((n - 1) // 2, n // 2))
        return 0.5 * (float(lo) + float(hi)), n

    keep = counts > 0
    sig, used, it = float("nan"), 0, 0
    while (counts[keep]).sum() > 0 and it < steps:
        m, used = middle(values[keep], counts[keep])
        sig = 1.4826 * middle(np.abs(values[keep] - m), counts[keep])[0]
        it += 1
        new = (counts > 0) & (np.abs(values - m) <= kappa * sig)
        if (new == keep).all():
            break
        keep = new
    return sig, used, it


def _counts(img):
    """Sorted finite FP16 values and the number of pixels of each."""
    import torch
    total = torch.zeros(65536, dtype=torch.int64, device="cuda")
    flat = img.view(-1).view(torch.int16)
    for part in flat.split(1 << 28):
        total += torch.bincount(part.long() + 32768, minlength=65536)
    values = (np.arange(65536) - 32768).astype(np.int16).view(np.float16).astype(np.float64)
    counts = total.cpu().numpy()
    ok = np.isfinite(values)
    order = np.argsort(values[ok], kind="stable")
    return values[ok][order], counts[ok][order]


def _image(n, kind):
    import torch
    x = torch.empty((1, n), dtype=torch.float16, device="cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(n % 1000 + len(kind))
    for i, part in enumerate(x.view(-1).split(1 << 27)):
        z = torch.randn(part.numel(), generator=g, device="cuda")
        if kind == "two_scales":  # every other run of pixels a thousand times narrower
            z *= 1e-3 if i % 2 else 1.0
        else:
            z[torch.rand(part.numel(), generator=g, device="cuda") < 0.01] = float("nan")
        part.copy_(z)
    return x


@pytest.mark.parametrize("kind", ["masked", "two_scales"])
def test_counts_past_32_bits(kind):
    import torch
    import paper_2503_08854_amd as dt
    ctx = dt.Context(0)
    small = _image(100003, kind)
    assert _mad_of_counts(*_counts(small), 3.0, 10) == oracle.mad_noise(small.float().cpu().numpy(), 3.0, 10)
    big = _image((1 << 32) + (1 << 27) + 123457, kind)  # finite ones past 2^32 too
    want = [_mad_of_counts(*_counts(x), 3.0, 10) for x in (big, small)]
    sig, used, it = dt.image_noise(ctx, [big, small], 3.0, 10)
    torch.cuda.synchronize()
    assert used.cpu().tolist() == [w[1] for w in want]
    assert it.cpu().tolist() == [w[2] for w in want]
    assert sig.cpu().tolist() == [w[0] for w in want]
    ctx.close()
