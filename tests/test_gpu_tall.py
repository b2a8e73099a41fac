"""Matched-filter planes of an image one column wide with nearly 2^31 rows,
where 32-bit row arithmetic overflows: pieces of the plane at both ends and in
between equal the definition's, to the rounding of FP32 sums (each value is a
sum of 2R + 1 products: 2 (2R + 3) + 4 roundings of the sum of magnitudes)."""
import math

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

H = 2147483000


def test_plane_of_the_tallest_column():
    import torch
    import paper_2503_08854_amd as dt
    if torch.cuda.get_device_properties(0).total_memory < 60e9:
        pytest.skip("needs 45 GB of device memory")
    fwhm = 3.0
    R = math.ceil(3 * fwhm / (2 * math.sqrt(2 * math.log(2))))
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    d, v = (torch.empty((H, 1), dtype=torch.float16, device="cuda") for _ in range(2))
    for a, b in zip(d.split(1 << 28), v.split(1 << 28)):
        a.copy_(torch.randn(a.shape, generator=g, device="cuda"))
        b.copy_(0.5 + torch.rand(b.shape, generator=g, device="cuda"))
    exps = [dict(t=1.0, obs=[1.0, 0.0, 0.0], crval=[10.0, 5.0], crpix=[1.0, 1.0], cd=[-5e-5, 0.0, 0.0, 5e-5], width=1,
                 height=H, fwhm=fwhm)]
    ctx = dt.Context(0)
    patch = dt.Patch(ctx, exps, [d], [v])
    got = patch.plane(0)
    tol = (2 * (2 * R + 3) + 4) * 2.0 ** -24
    for y0 in (0, 1 << 20, (1 << 30) - 300, 2130706433 - 300, H - 600):
        lo, hi = max(y0 - R, 0), min(y0 + 600 + R, H)
        dh, vh = d[lo:hi].cpu().numpy(), v[lo:hi].cpu().numpy()
        psi, phi = oracle.planes(dh, vh, fwhm)
        mag, _ = oracle.planes(np.abs(dh), vh, fwhm)
        at = slice(y0 - lo, y0 - lo + 600)
        part = got[y0:y0 + 600].cpu().numpy().astype(np.float64)
        assert (np.abs(part[..., 0] - psi[at]) <= tol * mag[at] + 1e-30).all(), y0
        assert (np.abs(part[..., 1] - phi[at]) <= tol * phi[at] + 1e-30).all(), y0
    patch.close()
    ctx.close()
